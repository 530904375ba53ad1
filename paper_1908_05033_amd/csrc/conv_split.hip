// dsq_conv2d for layers of few output tiles: one image, or a few, of a small map.  The
// LDS-patch kernel gives such a layer a handful of workgroups (512 -> 512 at 7x7: eight, on 256
// compute units), each of which walks the whole dot product, nine taps of every 64-channel
// block, stage by stage.
//
// Here a workgroup of eight waves owns a tile of 32 pixels x 32 channels (four times as many
// workgroups and more) and splits its dot product, a step being one tap of one channel block:
// wave w multiplies steps w*per .. w*per+per-1, the loads of U steps in flight together,
// operands straight from global memory (weights are in lane order; a lane reads 8 bytes
// of its own pixel's row, from L2: there are few of them).  The eight partial tiles meet in LDS
// (integer adds: exact in any order) and four waves run the shared dequantizing epilogue, or the next layer's
// quantizer, on a quarter of the tile each.  Formats, arithmetic and epilogue are those of the
// other kernels, and so are the results, bit for bit.
//
// Bound by latency: launch, one round trip for a wave's steps, the sum, the stores.
#include "conv_epilogue.h"
#include "patch_plan.h"

namespace {

constexpr int SPLIT_WAVES = 8;

struct SplitPlan {
    int tiles_m, total, xcd_chunk, per;             // pixel tiles, tiles, tiles per XCD, steps per wave
    uint32_t mg_tiles_m, mg_Wo, mg_Ho;              // division constants (see dsq_idiv)
};

// Compile-time forms, so that the registers of one are not those of all: two workgroups of up to
// 128 registers share a compute unit (nine steps of 4 bits in flight pass that: the layers that have
// them keep to one; with the tap sums of l_a != 0 in one kernel with the
// rest, 128 -> 128 3x3 at 28x28 x 4 took 6.5 us for 4.7).
enum { SPLIT_PLAIN = 0, SPLIT_LA = 1, SPLIT_CODES = 2 };       // fp32 results, the same with l_a != 0, chained mode

template <int CONT, int U, int MODE>
__global__ __launch_bounds__(64 * SPLIT_WAVES) __attribute__((amdgpu_waves_per_eu(MODE == SPLIT_LA || (CONT == 4 && U == 9) ? 2 : 4))) void conv_split_kernel(DsqConvArgs a, SplitPlan pl)
{
    constexpr int KB_BYTES = 64 * CONT / 8;         // one pixel's 64-channel block
    __shared__ v4i part[SPLIT_WAVES * 4 * 64];      // [wave][group of four channels][lane]
    __shared__ uint32_t exch[MODE == SPLIT_CODES ? 2 * 4 * 64 : 1];        // chained mode: packed codes and code sums of four waves

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int col = lane & 31, h = lane >> 5;
    // (one batch of argument fetches instead of several round trips one after the other)
    asm volatile("" ::"s"(a.N), "s"(a.C_in), "s"(a.H), "s"(a.W), "s"(a.C_out), "s"(a.R), "s"(a.stride), "s"(a.pad), "s"(a.Ho),
                 "s"(a.Wo), "s"(a.Cp), "s"(a.act), "s"(a.pix_sum), "s"(a.wq), "s"(a.delta_w), "s"(a.l_w), "s"(a.out),
                 "s"(pl.tiles_m), "s"(pl.total), "s"(pl.xcd_chunk), "s"(pl.per), "s"(pl.mg_tiles_m), "s"(pl.mg_Wo), "s"(pl.mg_Ho));
    // Workgroups are dealt to the 8 XCDs in turn: the pixel tiles of a channel tile run on one, so
    // that its weights are read into one L2
    const int logical = ((int)blockIdx.x & 7) * pl.xcd_chunk + ((int)blockIdx.x >> 3);
    if (logical >= pl.total) return;
    int mt;
    const int ct = dsq_idiv(logical, pl.tiles_m, pl.mg_tiles_m, mt);       // 32-channel tile: ct*32 < Cop
    const int M = a.N * a.Ho * a.Wo, m = mt * 32 + col;
    const int T = a.R * a.R, S = a.Cp / 64 * T;
    const int s0 = wave * pl.per, s1 = min(S, s0 + pl.per);

    // the lane's pixel, and which of its taps lie inside the image
    DsqPixel px;
    px.valid = m < M;
    px.n = dsq_idiv(dsq_idiv(px.valid ? m : 0, a.Wo, pl.mg_Wo, px.ox), a.Ho, pl.mg_Ho, px.oy);
    const int iy0 = px.oy * a.stride - a.pad, ix0 = px.ox * a.stride - a.pad;
    const int pixel0 = (px.n * a.H + iy0) * a.W + ix0;                     // tap 0 (used where it is inside)
    px.tapmask = 0;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        const bool in = px.valid && t < T && (unsigned)(iy0 + t / 3) < (unsigned)a.H && (unsigned)(ix0 + t % 3) < (unsigned)a.W;
        px.tapmask |= (in ? 1 : 0) << t;
    }
    px.ntaps = __builtin_popcount((unsigned)px.tapmask);

    const uint32_t row_bytes = (uint32_t)a.Cp * CONT / 8;
    const char *wq = (const char *)a.wq + (size_t)ct * S * 1024;
    v16i acc;
    v16f facc;
#pragma unroll
    for (int r = 0; r < 16; ++r) { acc[r] = 0; facc[r] = 0.f; }
    // channel block and tap of the wave's first step
    int cb = 0, t = 0;
    if (a.R == 3) { cb = s0 / 9; t = s0 - 9 * cb; } else cb = s0;
    // What the epilogue needs of its channels o0..o0+3 and its pixel, read behind the first steps'
    // loads (after the sum of the partial tiles everyone would wait for it).  Chained mode reads
    // its many constants there all the same: with them here 64 -> 512 3x3 at 7x7 x 1 6.3 us, without 5.7.
    const int o0 = ct * 32 + 8 * (wave & 3) + 4 * h;
    float4 dw = make_float4(0.f, 0.f, 0.f, 0.f), lw = dw;
    v4i sw = {0, 0, 0, 0};
    auto side_tables = [&] {
        int v[9];
#pragma unroll
        for (int k = 0; k < 9; ++k)                                        // (bits from T on are 0)
            v[k] = a.pix_sum[px.tapmask >> k & 1 ? pixel0 + k / 3 * a.W + k % 3 : 0];
        if (MODE != SPLIT_CODES) {
            dw = *reinterpret_cast<const float4 *>(a.delta_w + o0);
            lw = *reinterpret_cast<const float4 *>(a.l_w + o0);
        }
        if (MODE == SPLIT_LA && a.R == 1) {
            sw = px.tapmask & 1 ? *reinterpret_cast<const v4i *>(a.sw_tap + o0) : sw;
        } else if (MODE == SPLIT_LA) {
            int w[36];                                                     // nine taps of each of the four channels
#pragma unroll
            for (int k = 0; k < 9; ++k) {
                const v4i x = *reinterpret_cast<const v4i *>(a.sw_tap + (size_t)o0 * 9 + 4 * k);
                w[4 * k] = x.x; w[4 * k + 1] = x.y; w[4 * k + 2] = x.z; w[4 * k + 3] = x.w;
            }
            int n[4] = {0, 0, 0, 0};
#pragma unroll
            for (int k = 0; k < 36; ++k) n[k / 9] += px.tapmask >> (k % 9) & 1 ? w[k] : 0;
            sw = (v4i){n[0], n[1], n[2], n[3]};
        }
        px.sa = 0;
#pragma unroll
        for (int k = 0; k < 9; ++k) px.sa += px.tapmask >> k & 1 ? v[k] : 0;
    };
    for (int base = s0; base < s1; base += U) {
        v4i wf[U], af[U];
        uint32_t inside = 0;
#pragma unroll
        for (int i = 0; i < U; ++i) {
            // (never under a branch: past the last step that one comes again and is not multiplied)
            wf[i] = *reinterpret_cast<const v4i *>(wq + (size_t)min(base + i, s1 - 1) * 1024 + lane * 16);
            const int r = a.R == 3 ? (t * 11) >> 5 : 0, s = t - 3 * r;     // t / 3 for t < 9
            const bool in = px.tapmask >> t & 1;
            inside |= (in ? 1u : 0u) << i;
            const char *p = (const char *)a.act + (size_t)cb * KB_BYTES +
                            ((in ? (uint32_t)(pixel0 + r * a.W + s) * row_bytes : 0u) + 8u * (uint32_t)h);
            const v2i lo = *reinterpret_cast<const v2i *>(p);
            v2i hi = {0, 0};
            if (CONT == 4) hi = *reinterpret_cast<const v2i *>(p + 16);
            af[i] = (v4i){lo.x, lo.y, hi.x, hi.y};
            if (base + i + 1 < s1 && ++t == T) { t = 0; ++cb; }
        }
        if (base == s0 && wave < 4) side_tables();
#pragma unroll
        for (int i = 0; i < U; ++i) {
            if (base + i >= s1) continue;                                  // (uniform)
            const v4i x = inside >> i & 1 ? af[i] : (v4i){0, 0, 0, 0};
            if (CONT == 4) {
                // K halves: channels 32*kh + 16*h .. +15
                acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(dsq_unpack16_c4((v2i){wf[i].x, wf[i].y}),
                                                            dsq_unpack16_c4((v2i){x.x, x.y}), acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(dsq_unpack16_c4((v2i){wf[i].z, wf[i].w}),
                                                            dsq_unpack16_c4((v2i){x.z, x.w}), acc, 0, 0, 0);
            } else {
                facc = dsq_mfma_fp4(wf[i], dsq_fp4_from_c2((uint32_t)x.x, (uint32_t)x.y), facc);
            }
        }
    }
    if (CONT == 2) acc = dsq_fp4_acc_to_int(facc);
#pragma unroll
    for (int q = 0; q < 4; ++q)
        part[(wave * 4 + q) * 64 + lane] = (v4i){acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
    // (a wave of the epilogue without a step of its own: 1x1 layers of up to 192 channels)
    if (wave < 4 && s0 >= s1) side_tables();
    __syncthreads();
    if (wave < 4) {
        v4i sum = part[wave * 64 + lane];
#pragma unroll
        for (int w = 1; w < SPLIT_WAVES; ++w) {
            const v4i p = part[(w * 4 + wave) * 64 + lane];
            sum.x += p.x; sum.y += p.y; sum.z += p.z; sum.w += p.w;
        }
        if (MODE != SPLIT_CODES) {
            float y[4];
            const float dwv[4] = {dw.x, dw.y, dw.z, dw.w}, lwv[4] = {lw.x, lw.y, lw.z, lw.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                double v = dsq_terms(px, sum[j], a.delta_a, dwv[j], lwv[j]);
                if (MODE == SPLIT_LA && a.l_a != 0.0f) v += dsq_terms_la(a, px, dwv[j], lwv[j], sw[j]);
                y[j] = (float)v;
            }
            dsq_store4_of(a, px, m, o0, sum, y);
        } else {
            const int top_n = (1 << a.rq_bits) - 1;
            int codes = 0;
            exch[wave * 64 + lane] = dsq_requant_quarter<SUMS_FIRST>(a, px, o0, sum, a.delta_a, dsq_delta(a.rq_l, a.rq_u, top_n), top_n, codes);
            exch[(4 + wave) * 64 + lane] = (uint32_t)codes;
        }
    }
    if (MODE != SPLIT_CODES) return;
    // chained mode: a lane pair of one wave holds whole packed words of its pixel, so the
    // quarters meet in LDS and wave 0 packs, stores and adds to the pixel sums
    __syncthreads();
    if (wave == 0) {
        uint32_t bytes[4];
        int codes = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            bytes[q] = exch[q * 64 + lane];
            codes += (int)exch[(4 + q) * 64 + lane];
        }
        const int total = dsq_requant_store32(a, px.valid ? m : -1, ct * 32, h, bytes, codes);
        if (h == 0 && px.valid) atomicAdd(a.rq_pix + m, total);
    }
}

long long split_tiles(const DsqConvArgs &a)
{
    return (((long long)a.N * a.Ho * a.Wo + 31) / 32) * (((a.rq ? a.rq_Cp : a.C_out) + 31) / 32);
}

}  // namespace

// Up to a tile per compute unit it is ahead of the LDS-patch kernel on every layer measured (us, that kernel / this
// one, operands in the last-level cache: 64 -> 64 3x3 at 32x32 x 1 4.5 / 3.4, 128 -> 128 at 28x28 x 2 6.0 / 3.7, 512 -> 512 at
// 7x7 x 1 10.6 / 7.1, 2 bits 8.8 / 5.3, 512 -> 512 stride 2 at 7x7 x 32 19.3 / 7.2, 300 -> 90 at 20x20 x 1
// 9.3 / 4.9).  With two tiles a unit the patch's re-use of the activations begins to tell: stride 2, where a
// patch holds four times the pixels, stays ahead (64 -> 64 at 56x56 x 8 6.3 / 4.8), stride 1 where the dot
// product is short (128 -> 128 at 28x28 x 4 6.1 / 4.7; 256 -> 256 at 14x14 x 8 2 bits 6.7 / 5.6, but 4 bits
// 7.5 / 9.2); from 600 tiles on it falls behind (9.8 / 10.7 for 300 -> 90 at 20x20 x 16, then 1.2 to 3 times).
// Chained layers add to pixel sums that a launch of its own has to clear first (2.4 us), which the patch kernel
// does without where a workgroup holds all channels: up to 64 of them only the deepest dot products pay for
// that (512 -> 64 at 14x14 x 1 11.0 / 9.7; 64 -> 64 at 32x32 x 1 5.2 / 5.7), and none whose caller clears
// the sums: the patch kernel stores them whatever they hold.  (With l_a != 0 it does not take chained layers.)
// (Not where the caller has several calls in flight: they fill the chip together, and this kernel reads
// activations once per tap and channel tile.)
bool dsq_conv_split_preferred(const DsqConvArgs &a)
{
    if (a.cont == 3 || a.many_in_flight) return false;
    const int S = a.Cp / 64 * a.R * a.R;
    if (a.rq && a.l_a == 0.0f && a.C_out <= 64 && (a.rq_zeroed || S < 72)) return false;
    const long long tiles = split_tiles(a);
    return tiles <= 256 || (tiles <= 512 && (a.l_a == 0.0f || a.rq) && ((a.R == 3 && a.stride == 2) || S * (a.cont == 4 ? 2 : 1) <= 36));
}

hipError_t dsq_launch_conv_split(const DsqConvArgs &a, hipStream_t stream)
{
    const int M = a.N * a.Ho * a.Wo, S = a.Cp / 64 * a.R * a.R;
    SplitPlan pl;
    pl.tiles_m = (M + 31) / 32;
    pl.total = (int)split_tiles(a);
    pl.xcd_chunk = (pl.total + 7) / 8;
    pl.per = (S + SPLIT_WAVES - 1) / SPLIT_WAVES;
    pl.mg_tiles_m = dsq_division_constant(pl.tiles_m);
    pl.mg_Wo = dsq_division_constant(a.Wo);
    pl.mg_Ho = dsq_division_constant(a.Ho);
    // chained mode: the channel tiles add to the next layer's pixel sums, which a fill kernel
    // clears first unless the caller did (no memset node: the call may be under graph capture)
    if (a.rq && !a.rq_zeroed) {
        const hipError_t e = dsq_launch_fill_zero(a.rq_pix, (size_t)M, stream);
        if (e != hipSuccess) return e;
    }
    const int grid = 8 * pl.xcd_chunk;
    const int mode = a.rq ? SPLIT_CODES : a.l_a != 0.0f ? SPLIT_LA : SPLIT_PLAIN;
#define DSQ_SPLIT_U(CONT, U) \
    do { \
        if (mode == SPLIT_PLAIN) conv_split_kernel<CONT, U, SPLIT_PLAIN><<<grid, 64 * SPLIT_WAVES, 0, stream>>>(a, pl); \
        else if (mode == SPLIT_LA) conv_split_kernel<CONT, U, SPLIT_LA><<<grid, 64 * SPLIT_WAVES, 0, stream>>>(a, pl); \
        else conv_split_kernel<CONT, U, SPLIT_CODES><<<grid, 64 * SPLIT_WAVES, 0, stream>>>(a, pl); \
    } while (0)
#define DSQ_SPLIT(CONT) \
    do { if (pl.per <= 3) DSQ_SPLIT_U(CONT, 3); else if (pl.per <= 6) DSQ_SPLIT_U(CONT, 6); else DSQ_SPLIT_U(CONT, 9); } while (0)
    if (a.cont == 4) DSQ_SPLIT(4); else DSQ_SPLIT(2);
#undef DSQ_SPLIT
#undef DSQ_SPLIT_U
    return hipGetLastError();
}
