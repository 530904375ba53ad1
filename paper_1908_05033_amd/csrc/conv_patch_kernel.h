// dsq_conv2d, LDS-patch kernel (the tuned path).
//
// GEMM view of Algorithm 1 step 5 of the paper: rows = output channels,
// columns = output pixels, K = filter taps x input channels, run on
// v_mfma_i32_32x32x32_i8 with int32 accumulation (the integer-arithmetic
// deployment of Sec. 3.5 / 4.5, re-designed for the matrix cores; the
// 16x16x64 form of the instruction issues at half the rate on this chip).
//
// A workgroup (4 wavefronts, WP x WC) owns BP = 32*PF*WP consecutive output
// pixels of a strip of TW output columns (pixels are numbered row by row
// through the whole batch, so a tile may span rows and images) and
// BC = 32*CT*WC output channels; a wavefront owns PF fragments of 32 pixels and
// CT tiles of 32 channels.  K is walked in stages of 64 input channels.  For a
// stage, the input patch that all R*R taps of the tile touch is read from
// HBM/L2 once, unpacked from 2/4-bit codes to int8 and kept in LDS; the taps
// then read shifted windows of it, so the R*R-fold re-use of the activations
// never leaves the CU.  Positions of the patch that fall in the zero padding
// hold code 0: they add nothing to the integer sums, and the epilogue's SA /
// SW / KV terms leave them out as well.  Weight fragments were laid out per
// lane by dsq_pack_weights and go from global memory straight to registers,
// each refilled for the next stage right after its use.  The patch of the next
// stage is fetched while the current one is multiplied (two LDS buffers, one
// barrier per stage).
//
// Feed rates that shape the tiles (measured on MI355X): LDS delivers 128 B/clk
// per CU, the vector L1 one wave-wide load (<= 16 B per lane) per 16 clk per
// CU.  With 4 waves issuing MFMAs back to back, activation fragments keep the
// LDS busy 1/CT of the time and weight fragments keep the L1 busy 1/PF of the
// time.
#pragma once
#include <type_traits>

#include "conv_epilogue.h"
#include "patch_plan.h"

struct PatchPlan {
    int TW;            // strip width in output columns
    int BP;            // pixels per tile
    int tiles_w;       // strips per output row
    int row_tiles;     // tiles per strip
    int PR, PC;        // patch rows (max over tiles) x patch columns
    int RP;            // LDS bytes per patch row
    int buf_bytes;     // LDS bytes of one patch buffer (incl. a 64-byte dump slot at its end)
    int Hp;            // H + 2*pad: rows of one image in the padded row space
    int units;         // 16-byte fetch units per stage
    int aux_off;       // LDS offset of the small tables that follow the patch / staging area
    int tiles_c;       // channel tiles (workgroups per pixel tile)
    int total_blocks;  // pixel tiles * channel tiles
    int xcd_chunk;     // ceil(total_blocks / 8)
    uint32_t mg_tiles_c;   // division constants (see dsq_idiv) of tiles_c ...
    int step_q, step_r;   // (256 / units-per-pixel) divided by PC: quotient and remainder
    uint32_t mg_PC, mg_TW, mg_Hp, mg_Ho, mg_tiles_w;   // ... and of PC, TW, Hp, Ho, tiles_w
};

namespace {

// LDS bytes per patch pixel: 64 int8 (4-bit containers) or 32 bytes of FP4
// nibbles (2-bit) plus padding that makes the stride an odd multiple of 16, so
// that the 16-byte reads of 16 consecutive pixels fall into distinct bank groups.
constexpr int pix_stride(int cont) { return cont == 2 ? 48 : 80; }


// Workgroup barrier that orders LDS traffic only.  __syncthreads() also drains
// the vector-memory counter, which would expose the latency of the global
// loads that are deliberately left in flight across stage boundaries.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Chained mode, per output channel o: the constants of the code-unit form of the
// layer-to-layer map.  With P = Da*Dw[o], Q = Da*l_w[o], scale sc and shift sh, the real
// value of the next layer's input in units of its quantizer step, counted from l_n, is
//   T = ((P*ACC + Q*SA)*sc + sh - l_n)/D_n = A*(ACC + rho*SA) + s,
//   A = P*sc/D_n, rho = Q/P = l_w/Dw, s = sh/D_n + c0, c0 = -l_n/D_n,
// and the code is T rounded to the nearest integer, clamped to the code range.  The kernel
// evaluates
//   u = fma(SA, rho32, ACC)             one rounding, of the small difference: the two
//                                       large terms cancel inside the fma
//   T = fma(u, A32, fma(SA, B32, s32))  B = A*(rho - rho32): the part of rho that
//                                       binary32 drops
// The exact sequence (fp32 value of the layer, times scale, plus shift: three
// roundings) and this one (three roundings, four rounded constants) each differ from
// the real T by a few 2^-24 of |T| + S, S = |sh|/D_n + |c0| + 1, in total less than
//   E = 2^-21*(2^bits + S) + 2^-45*|Q*sc/D_n|*SA_max
// for T inside the code range (6|T| + 7S times 2^-24 to first order; the last term
// covers the rounding of B and of the fma that uses it).  Outside the range both
// clamp alike when E < 1/2.  Returns how far T must stay from every half-integer for its
// nearest integer to be the exact sequence's code: E plus what the host adds for the
// quantizer's own roundings (DsqConvArgs); 1 (never) for channels whose magnitudes
// would let an intermediate of either sequence overflow, or lose bits to denormals, and
// when the host disabled the form: those keep harmless constants, so that T stays
// finite.  Channels past C_out get constants that give code 0 safely (T = 0, half a step from the nearest
// half-integer; their bytes are blanked anyway), and a distance of 0: the workgroup's is the largest of its channels'.
//
// A wave computes the constants of 64 channels before the main loop, in binary32 but for A
// and s: rho32 is the quotient corrected by its remainder, r the remainder of that,
// r/Dw = rho - rho32 to 22 bits.  (With a binary64 division, after the main loop where every
// wave waits for it, the constants took 1400 clocks of a workgroup's 24000.)
//
// `unit`: the kernel's accumulators hold ACC/unit (the FP4 form counts in quarter
// units): A*unit and rho32/unit are stored, both exact scalings by a power of two.
__device__ __forceinline__ float chained_channel_constants(const DsqConvArgs &a, bool real, float dw, float lw, float sc,
                                                           float sh, float unit, float4 &k)
{
    k = make_float4(0.f, 0.f, 0.f, 0.f);
    float y = __builtin_amdgcn_rcpf(dw);
    y = __builtin_fmaf(__builtin_fmaf(-dw, y, 1.0f), y, y);
    float rho = lw * y;
    rho = __builtin_fmaf(__builtin_fmaf(-rho, dw, lw), y, rho);
    const float rest = __builtin_fmaf(-rho, dw, lw) * y;
    const float A = (float)((double)dw * (double)sc * a.rq_da_dn);
    const float s = (float)__builtin_fma((double)sh, a.rq_inv_dn, a.rq_c0);
    const float inv_dn = (float)a.rq_inv_dn, c0 = __builtin_fabsf((float)a.rq_c0), samax = a.rq_sa_max;
    const float S = __builtin_fabsf(sh) * inv_dn + c0 + 1.0f, q = __builtin_fabsf(a.delta_a * lw);
    // (1.001: the roundings of the bound itself)
    const float E = 1.001f * (0x1p-21f * ((float)(1 << a.rq_bits) + S) + 0x1p-45f * (q * __builtin_fabsf(sc)) * inv_dn * samax) + a.rq_t_slack;
    const float ymax = (__builtin_fabsf(a.delta_a * dw) * a.rq_w_max + q) * samax;               // bound on the layer's |output|
    // (every comparison is false for a NaN, which then ends in 1.  Dw is bounded above as well: from 2^126 on
    // its reciprocal is a denormal, which v_rcp_f32 returns as 0, and rho with it)
    const bool ok = a.rq_fast && dw >= 0x1p-80f && dw < 0x1p100f && __builtin_fabsf(lw) < 0x1p100f && ymax < 0x1p100f &&
                    ymax * __builtin_fabsf(sc) < 0x1p100f && __builtin_fabsf(sh) < 0x1p100f &&
                    (__builtin_fabsf(sc) + 1.0f) * inv_dn < 0x1p100f && __builtin_fabsf(A) < 0x1p60f &&
                    __builtin_fabsf(rho) < 0x1p20f && E < 0.5f;
    if (!real) return 0.0f;
    if (!ok) return 1.0f;
    k = make_float4(A * unit, rho / unit, A * rest, s);
    return E;
}

// Which of the three taps from row (column) i on lie inside an image of n rows: 0 all, 1 all but
// the first, 2 all but the last, 3 the last, 4 the first; 0 as well where n = 1 and i = -1, whose pixels have
// the middle tap only.  (3 and 4 with two rows of padding only.)
__device__ __forceinline__ int border_class(int i, int n)
{
    return i < -1 ? 3 : i > n - 2 ? 4 : n == 1 ? 0 : i < 0 ? 1 : i + 2 >= n ? 2 : 0;
}

// What the kernel's results become; chosen at compile time, so that the register
// allocation of each epilogue is its own.
//   OUT_PLAIN    fp32 NHWC tensor, l_a = 0, C_out a multiple of 4, no raw accumulators
//   OUT_CODES    the next layer's codes (chained mode)
//   OUT_ROWS     fp32 NHWC tensors of any C_out and l_a, a lane holding a channel instead of a pixel
//   OUT_GENERAL  everything else: NCHW, l_a != 0 (terms that depend on which taps lie
//                inside the image), raw accumulators
enum { OUT_PLAIN = 0, OUT_CODES = 1, OUT_GENERAL = 2, OUT_ROWS = 3 };

// Two rows of padding and l_a != 0: 25 classes of borders instead of 9, in a table of their own.
__host__ __device__ inline bool has_wide_border(const DsqConvArgs &a) { return a.l_a != 0.0f && a.pad == 2; }
constexpr int wide_table_bytes(int BC) { return 25 * BC * 8; }

// BC: channels of the workgroup's tile.  OUT_ROWS where C_out is not a multiple of 4 (single floats
// are staged badly: 64 -> 66 3x3 at 56x56 x 8 9.5 us, 8.0 so) and for 1x1 layers with l_a != 0 a fifth of
// whose tiles' channels or more do not exist (it leaves those out: 24 -> 144 at 56x56 x 64 37.4 and 32.7 us,
// 144 -> 24 14.6 and 14.2); the other way round without that (320 -> 1280 at 7x7 x 64 8.2 and 8.6) and
// on 3x3 layers (64 -> 64 at 56x56 x 64 19.2 and 20.7).
inline int output_mode(const DsqConvArgs &a, int BC)
{
    if (a.rq) return OUT_CODES;
    if (a.out_nchw || a.acc != nullptr) return OUT_GENERAL;
    if ((a.C_out & 3) != 0) return OUT_ROWS;
    if (a.l_a == 0.0f) return OUT_PLAIN;
    const int padded = (a.C_out + BC - 1) / BC * BC;
    return a.R == 1 && 5 * (padded - a.C_out) >= padded ? OUT_ROWS : OUT_GENERAL;
}

template <int CONT, int R, int WP, int WC, int PF, int CT, int UPT, int WD, int OCC, int KS, int OUT>
__global__ __launch_bounds__(256 * KS) __attribute__((amdgpu_waves_per_eu(OCC, OCC))) void conv_patch_kernel(DsqConvArgs a, PatchPlan pl)
{
    constexpr int T = R * R;
    constexpr bool RQ = OUT == OUT_CODES;
    // CONT: 2 / 4 = container width of the packed activation codes, 3 = dense 3-bit units
    // (12 bytes per 32 channels; everything after the patch store is the 4-bit path)
    constexpr int UPP = CONT == 2 ? 1 : 2;        // fetch units per patch pixel and 64 channels
    constexpr int UNIT_B = CONT == 3 ? 12 : 16;   // bytes of a fetch unit
    constexpr int KB_BYTES = 64 * CONT / 8;       // packed bytes of 64 channels
    constexpr int WLANE = 16;                     // weight bytes per lane per (tile, cb, tap)
    constexpr bool F4 = CONT == 2;                // 2-bit layers run on the FP4 matrix instruction
    constexpr int KH = F4 ? 1 : 2;                // matrix instructions per 64 channels
    constexpr int PIX_STRIDE = pix_stride(CONT);
    static_assert(WP * WC == 4, "four waves per workgroup");
    static_assert(64 * CT * WC <= 256, "one thread per staged channel constant");
    typedef v4i wpack_t;
    typedef typename std::conditional<F4, v16f, v16i>::type macc_t;   // main-loop accumulator

    extern __shared__ __attribute__((aligned(16))) char lds[];
    // LDS: [patch buffer 0][patch buffer 1] (re-used by the epilogue as staging)
    //      at aux_off: [double Da*Dw[BC]][double Da*l_w[BC]]
    //                  [int pixel code sums of the patch, PR*PC]
    constexpr int BC = 32 * CT * WC;
    double *pq_lds = reinterpret_cast<double *>(lds + pl.aux_off);
    int *pix_lds = reinterpret_cast<int *>(pq_lds + 2 * BC);
    // chained mode: in the place of the binary64 tables (Dw, l_w, scale, shift) of the
    // workgroup's channels; behind the code sums, 16-byte aligned, the constants (A, rho, B, s)
    // of the code-unit form, and per 64 channels the distance from a half-integer at which
    // every channel's code is safe
    float4 *raw_lds = reinterpret_cast<float4 *>(pq_lds);
    float4 *ft_lds = reinterpret_cast<float4 *>(lds + ((pl.aux_off + 2 * BC * 8 + pl.PR * pl.PC * 4 + 15) & ~15));
    float *te_lds = reinterpret_cast<float *>(ft_lds + BC);
    // results of a layer with l_a != 0 (in the place of the chained mode's tables): the border
    // terms l_a*Dw*SW + KV*l_a*l_w of the workgroup's channels, [class][channel], a class for each of
    // the sets of taps that lie inside the image (see border_class)
    double *wt_lds = reinterpret_cast<double *>(ft_lds);

    // KS = 2: two groups of four waves work on alternating 64-channel blocks of K
    // (each with its own patch buffers) and add their accumulators at the end, so
    // that every SIMD hosts two waves whose MFMA and VALU phases can overlap even
    // when the layer yields only one workgroup per CU.
    static_assert(KS == 1 || KS == 2, "one or two wave groups");
    const int tid = threadIdx.x & 255;                 // thread index inside its wave group
    const int lane = tid & 63;
    const int grp = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave index inside the group
    const int col = lane & 31, h = lane >> 5;
    const int wp = wave % WP, wc = wave / WP;

    // The kernel arguments live in memory that is slow to reach.  Naming all of
    // them as scalar-register inputs of an (empty) asm statement right here makes
    // the compiler fetch them in one batch at the top of the kernel -- one round
    // trip instead of one per group of first uses -- at no instruction cost.
    asm volatile("" ::"s"(a.N), "s"(a.C_in), "s"(a.H), "s"(a.W), "s"(a.C_out), "s"(a.stride), "s"(a.pad),
                 "s"(a.bits), "s"(a.Ho), "s"(a.Wo), "s"(a.Cp), "s"(a.out_nchw), "s"(a.R), "s"(a.Cop),
                 "s"(a.l_a), "s"(a.u_a), "s"(a.delta_a), "s"(a.act), "s"(a.pix_sum), "s"(a.wq), "s"(a.delta_w), "s"(a.l_w),
                 "s"(a.out), "s"(a.acc));
    asm volatile("" ::"s"(pl.TW), "s"(pl.BP), "s"(pl.tiles_w), "s"(pl.PR), "s"(pl.PC), "s"(pl.RP),
                 "s"(pl.buf_bytes), "s"(pl.Hp), "s"(pl.aux_off), "s"(pl.step_q), "s"(pl.step_r),
                 "s"(pl.tiles_c), "s"(pl.total_blocks), "s"(pl.xcd_chunk), "s"(pl.mg_tiles_c), "s"(pl.mg_PC),
                 "s"(pl.mg_TW), "s"(pl.mg_Hp), "s"(pl.mg_Ho), "s"(pl.mg_tiles_w));
    // (chained mode: the one cache line of them that the above does not touch)
    if (RQ) asm volatile("" ::"s"(a.rq_t_lo));

    // Workgroups are dealt round-robin to the 8 XCDs (each with its own L2).  Give
    // every XCD a contiguous range of tiles, channel tiles of one pixel tile
    // first, so that the tiles that share activations (same pixels, halo rows of
    // neighbours) meet in one L2.
    const int logical = ((int)blockIdx.x & 7) * pl.xcd_chunk + ((int)blockIdx.x >> 3);
    if (logical >= pl.total_blocks) return;
    int blk_y;
    const int blk_x = dsq_idiv(logical, pl.tiles_c, pl.mg_tiles_c, blk_y);

    const int NCB = a.Cp / 64;
    const int NHo = a.N * a.Ho;

    // ---- weights first: their addresses need only the lane and block ids ----
    // lane-ordered fragments, [ct][cb][tap][lane][both K halves]
    const int ct0 = (blk_y * WC + wc) * CT;
    const uint32_t lane_woff = (uint32_t)lane * WLANE;
    // Packed weight fragments travel WD taps ahead of their use in a ring of
    // registers (slot = tap % WD; WD divides the tap count); a slot is refilled as
    // soon as it has been unpacked.
    static_assert(T % WD == 0, "ring period must divide the taps of a stage");
    wpack_t wreg[CT][WD];
    auto fetch_weight = [&](int c, int t, int cb) {
        const char *p = (const char *)a.wq +
                        ((((size_t)(ct0 + c) * NCB + cb) * T + t) * 64) * WLANE + lane_woff;
        wreg[c][t % WD] = *reinterpret_cast<const wpack_t *>(p);
    };
    // (a group whose first channel block does not exist fetches block 0 and never uses it)
    const int cb_first = grp < NCB ? grp : 0;
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int t = 0; t < WD; ++t) fetch_weight(c, t, cb_first);


    // ---- tile position -------------------------------------------------------
    int tile_w;
    const int tile_r = dsq_idiv(blk_x, pl.tiles_w, pl.mg_tiles_w, tile_w);
    const int t0 = tile_r * pl.BP;              // first pixel of the tile, numbered inside the strip
    const int ow0 = tile_w * pl.TW;
    int tc0;
    const int gr0 = dsq_idiv(t0, pl.TW, pl.mg_TW, tc0);   // its output row (batch-wide numbering)
    int oh0;
    const int n0 = dsq_idiv(gr0, a.Ho, pl.mg_Ho, oh0);
    const int v0 = n0 * pl.Hp + oh0 * a.stride;   // first padded input row of the patch
    const int vc0 = ow0 * a.stride;               // first padded input column of the patch
    const uint32_t row_bytes = (uint32_t)a.Cp * CONT / 8;

    // ---- per-thread fetch units of the patch ---------------------------------
    // unit u = tid + 256*k covers half `u % UPP` of patch pixel u / UPP; (prow, pcol)
    // and the image row behind prow advance by fixed steps from unit to unit
    uint32_t src_off[UPT];   // byte offset into act of the unit at channel block 0
    uint32_t src_pix[UPT];   // index of the unit's input pixel (0 if none)
    int dst_off[UPT];        // LDS byte offset inside a patch buffer (dump slot if no such unit)
    uint32_t src_valid = 0;  // bit k: unit k reads real data (else: zero padding)
    const int dump_off = pl.buf_bytes - 64;
    const int half = UPP == 2 ? (tid & 1) : 0;
    {
        int pcol, ihp;
        int prow = dsq_idiv(UPP == 2 ? (tid >> 1) : tid, pl.PC, pl.mg_PC, pcol);
        int n = dsq_idiv(v0 + prow, pl.Hp, pl.mg_Hp, ihp);
#pragma unroll
        for (int k = 0; k < UPT; ++k) {
            const int ih = ihp - a.pad, iw = vc0 + pcol - a.pad;
            const bool inpatch = prow < pl.PR;
            const bool valid = inpatch && n < a.N && (unsigned)ih < (unsigned)a.H && (unsigned)iw < (unsigned)a.W;
            const uint32_t pix = valid ? (uint32_t)((n * a.H + ih) * a.W + iw) : 0u;
            src_pix[k] = pix;
            src_off[k] = pix * row_bytes + half * UNIT_B;
            dst_off[k] = inpatch ? prow * pl.RP + pcol * PIX_STRIDE + half * 32 : dump_off;
            src_valid |= (valid ? 1u : 0u) << k;
            int dp = pl.step_q;
            pcol += pl.step_r;
            if (pcol >= pl.PC) { pcol -= pl.PC; ++dp; }
            prow += dp;
            ihp += dp;
            while (ihp >= pl.Hp) { ihp -= pl.Hp; ++n; }  // seldom more than once
        }
    }

    v4i pre[UPT];            // packed patch units in flight
    auto fetch_patch = [&](int cb) {
        const char *base = (const char *)a.act + (size_t)cb * KB_BYTES;
#pragma unroll
        for (int k = 0; k < UPT; ++k) {
            if constexpr (CONT == 3) {
                typedef int v3i __attribute__((ext_vector_type(3)));
                const v3i t = *reinterpret_cast<const v3i *>(base + src_off[k]);      // (4-byte aligned)
                pre[k] = (v4i){t.x, t.y, t.z, 0};
            } else {
                pre[k] = *reinterpret_cast<const v4i *>(base + src_off[k]);
            }
        }
    };
    auto store_units = [&](char *buf, const v4i (&units)[UPT]) {
#pragma unroll
        for (int k = 0; k < UPT; ++k) {
            const v4i pk = (src_valid >> k & 1) ? units[k] : (v4i){0, 0, 0, 0};
            char *d = buf + dst_off[k];
            if (CONT == 3) {
                // 12 packed bytes = 32 channels -> 32 int8
                uint32_t g[8];
                dsq_unpack32_d3((uint32_t)pk.x, (uint32_t)pk.y, (uint32_t)pk.z, g);
                *reinterpret_cast<v4i *>(d) = (v4i){(int)g[0], (int)g[1], (int)g[2], (int)g[3]};
                *reinterpret_cast<v4i *>(d + 16) = (v4i){(int)g[4], (int)g[5], (int)g[6], (int)g[7]};
            } else if (CONT == 4) {
                // 16 packed bytes = 32 channels -> 32 int8
                *reinterpret_cast<v4i *>(d) = dsq_unpack16_c4((v2i){pk.x, pk.y});
                *reinterpret_cast<v4i *>(d + 16) = dsq_unpack16_c4((v2i){pk.z, pk.w});
            } else {
                // 16 packed bytes = 64 channels -> two K groups of 32 FP4 nibbles
                *reinterpret_cast<v4i *>(d) = dsq_fp4_from_c2((uint32_t)pk.x, (uint32_t)pk.y);
                *reinterpret_cast<v4i *>(d + 16) = dsq_fp4_from_c2((uint32_t)pk.z, (uint32_t)pk.w);
            }
        }
    };
    auto store_patch = [&](char *buf) { store_units(buf, pre); };
    fetch_patch(cb_first);
    // side tables, needed only after the main loop: the pixels' code sums and the
    // per-channel dequantization constants of this workgroup's channels
    int pix_val[UPT];
#pragma unroll
    for (int k = 0; k < UPT; ++k) pix_val[k] = a.pix_sum[src_pix[k]];
    // (every lane loads an entry, used or not: a load under a branch would drag
    // the wait for it, and for everything issued before it, up to this point)
    const int chan_i = tid < 2 * BC ? tid : 0;
    const int chan_o = blk_y * BC + (chan_i < BC ? chan_i : chan_i - BC);      // < Cop by construction
    float chan_const = 0.f;
    if (!RQ) chan_const = (chan_i < BC ? a.delta_w : a.l_w)[chan_o];
    // chained mode: step and level of the channels, scale and shift (one channel per thread)
    float4 raw = make_float4(0.f, 0.f, 0.f, 0.f);
    const int rq_o = blk_y * BC + (tid < BC ? tid : 0);
    if (RQ) {
        const int in = rq_o < a.C_out ? rq_o : 0;
        raw.x = a.delta_w[rq_o];
        raw.y = a.l_w[rq_o];
        raw.z = (a.rq_scale != nullptr ? a.rq_scale : a.delta_w)[in];
        raw.w = (a.rq_shift != nullptr ? a.rq_shift : a.delta_w)[in];
    }

    const bool has_la = (OUT == OUT_GENERAL || OUT == OUT_ROWS) && a.l_a != 0.0f;
    const bool wide = T > 1 && has_la && has_wide_border(a);
    // (one channel per thread; behind the patch, so that the wait for that is not one for these)
    int la_sw[T];
    float la_dw = 0.f, la_lw = 0.f;
#pragma unroll
    for (int t = 0; t < T; ++t) la_sw[t] = 0;
    if (has_la) {
        const int o = blk_y * BC + (tid < BC ? tid : 0);          // < Cop: the side tables cover it
        la_dw = a.delta_w[o];
        la_lw = a.l_w[o];
#pragma unroll
        for (int t = 0; t < T; ++t) la_sw[t] = a.sw_tap[(size_t)o * T + t];
        if (T == 1 && grp == KS - 1 && tid < BC)
            wt_lds[tid] = ((double)a.l_a * (double)la_dw) * (double)la_sw[0] + (double)a.C_in * ((double)a.l_a * (double)la_lw);
    }

    // ---- per-lane LDS offsets of the fragments' pixels -----------------------
    // Tile pixels past the end of the strip multiply patch pixel 0 and are
    // never stored.
    int frag_off[PF];       // byte offset of the pixel's first tap inside a patch buffer
    int frag_pp[PF];        // index of that patch pixel (prow*PC + pcol)
    int frag_m[PF];         // output pixel index n*Ho*Wo + oy*Wo + ox, or -1
    int frag_base[PF];      // general results, NCHW: element index of the pixel in channel 0
    int frag_cls[PF];       // l_a != 0: class of the set of taps that lie inside the image
#pragma unroll
    for (int f = 0; f < PF; ++f) {
        const int t = t0 + (wp * PF + f) * 32 + col;
        int tc;
        const int gr = dsq_idiv(t, pl.TW, pl.mg_TW, tc);
        const int ow = ow0 + tc;
        const bool ok = gr < NHo && ow < a.Wo;
        int prow = 0, pcol = 0;
        frag_base[f] = 0;
        frag_cls[f] = 0;
        if (ok) {
            int oh;
            const int n = dsq_idiv(gr, a.Ho, pl.mg_Ho, oh);
            prow = n * pl.Hp + oh * a.stride - v0;
            pcol = tc * a.stride;
            if (OUT == OUT_GENERAL || OUT == OUT_ROWS) {
                frag_base[f] = n * (a.C_out - 1) * (a.Ho * a.Wo) + gr * a.Wo + ow;
                if (T > 1 && has_la) {
                    const int ih = oh * a.stride - a.pad, iw = ow * a.stride - a.pad;
                    frag_cls[f] = (wide ? 5 : 3) * border_class(ih, a.H) + border_class(iw, a.W);
                }
            }
        }
        frag_m[f] = ok ? gr * a.Wo + ow : -1;
        frag_pp[f] = prow * pl.PC + pcol;
        frag_off[f] = prow * pl.RP + pcol * PIX_STRIDE + 16 * h;
    }

    macc_t macc[PF][CT];
    const macc_t zero16 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int f = 0; f < PF; ++f)
#pragma unroll
        for (int c = 0; c < CT; ++c) macc[f][c] = zero16;

    // One stage: all taps of 64 input channels.  HAS_NEXT: the weights and the
    // patch of stage next_cb are fetched / stored on the way.
    auto compute = [&](auto has_next, const char *buf, int cur_cb, int next_cb, char *nextbuf) {
        constexpr bool HAS_NEXT = decltype(has_next)::value;
        v4i af[2][PF][KH];
#pragma unroll
        for (int f = 0; f < PF; ++f)
#pragma unroll
            for (int kh = 0; kh < KH; ++kh)
                af[0][f][kh] = *reinterpret_cast<const v4i *>(buf + frag_off[f] + 32 * kh);
        // (keep these LDS reads first in the stage: their latency then runs under the
        // unpacking of the first weight fragments instead of in front of the first MFMA.
        // Only where registers are plentiful: the one-group variants spill under
        // this constraint.)
        if constexpr (KS == 2) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < T; ++t) {
            if (t + 1 < T) {
                const int tap_off = ((t + 1) / R) * pl.RP + ((t + 1) % R) * PIX_STRIDE;
#pragma unroll
                for (int f = 0; f < PF; ++f)
#pragma unroll
                    for (int kh = 0; kh < KH; ++kh)
                        af[(t + 1) & 1][f][kh] =
                            *reinterpret_cast<const v4i *>(buf + frag_off[f] + tap_off + 32 * kh);
            }
            v4i wf[CT][KH];
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const wpack_t wr = wreg[c][t % WD];
                if (F4) {
                    wf[c][0] = wr;                       // FP4 nibbles go to the matrix cores as they are
                    // (1x1 filters, two wave groups: the slot is refilled for the next stage right below.
                    // The copy is made here, where the weights have to be there anyway; left to itself the
                    // compiler loads into other registers and copies at the end of the stage, which waits
                    // for the load: 25088 -> 4096 x 512 at 2 bits 133 us, 111 so.  With one group it does
                    // not, and the copy costs 6 %)
                    if constexpr (T == 1 && KS == 2) asm volatile("" : "+v"(wf[c][0]));
                } else {
                    wf[c][0] = dsq_unpack16_c4((v2i){wr[0], wr[1]});
                    wf[c][KH - 1] = dsq_unpack16_c4((v2i){wr[2], wr[3]});
                }
                if (t + WD < T) fetch_weight(c, t + WD, cur_cb);
                else if (HAS_NEXT) fetch_weight(c, t + WD - T, next_cb);
            }
            // (the loads just issued stay in front of this tap's matrix instructions:
            // left to itself the scheduler sinks each weight load to right before its
            // use, WD taps later, which exposes the full load latency at every tap.  Not
            // where the patch prefetch or the 4-bit 256x128 tile holds many registers (the
            // variants then spill), not on the 4-bit 128x128 tile (measured 3 % slower), and
            // not with two wave groups, where it measured slower)
            if constexpr (UPT <= 4 && KS == 1 && !(CONT >= 3 && (PF == 4 || (PF == 2 && WP == 2)))) __builtin_amdgcn_sched_barrier(0);
            // consecutive MFMAs go to different accumulators
#pragma unroll
            for (int kh = 0; kh < KH; ++kh)
#pragma unroll
                for (int c = 0; c < CT; ++c)
#pragma unroll
                    for (int f = 0; f < PF; ++f) {
                        // (OUT_ROWS: pixels in the rows, a lane holds one channel of 16 of them)
                        if constexpr (F4 && OUT == OUT_ROWS)
                            macc[f][c] = dsq_mfma_fp4(af[t & 1][f][kh], wf[c][kh], macc[f][c]);
                        else if constexpr (OUT == OUT_ROWS)
                            macc[f][c] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[t & 1][f][kh], wf[c][kh], macc[f][c], 0, 0, 0);
                        else if constexpr (F4)
                            macc[f][c] = dsq_mfma_fp4(wf[c][kh], af[t & 1][f][kh], macc[f][c]);
                        else
                            macc[f][c] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wf[c][kh], af[t & 1][f][kh], macc[f][c], 0, 0, 0);
                    }
            // half way through the taps the next stage's patch has arrived:
            // unpack it into the other buffer while the matrix cores are busy
            if (HAS_NEXT && t == (T / 2)) store_patch(nextbuf);
        }
    };

    // patch buffers: [parity][group]
    auto patch_buf = [&](int parity) { return lds + (parity * KS + grp) * pl.buf_bytes; };
    // (have the fragment offsets computed here, under the latency of the patch
    // fetch, rather than after the barrier where nothing hides them)
#pragma unroll
    for (int f = 0; f < PF; ++f) asm volatile("" ::"v"(frag_off[f]), "v"(frag_pp[f]), "v"(frag_m[f]));
    // (likewise the zeroing of the accumulators, where registers are plentiful)
    if constexpr (KS == 2) {
#pragma unroll
        for (int f = 0; f < PF; ++f)
#pragma unroll
            for (int c = 0; c < CT; ++c) asm volatile("" : "+v"(macc[f][c]));
    }
    store_patch(patch_buf(0));
    if (grp == 0) {
        int pp = UPP == 2 ? (tid >> 1) : tid;
#pragma unroll
        for (int k = 0; k < UPT; ++k) {
            if (pp < pl.PR * pl.PC && half == 0) pix_lds[pp] = (src_valid >> k & 1) ? pix_val[k] : 0;
            pp += 256 / UPP;
        }
        // Da*Dw[o] and Da*l_w[o] of this workgroup's channels, in binary64
        const double da0 = (double)a.delta_a;
        if (!RQ && tid < 2 * BC) pq_lds[tid] = da0 * (double)chan_const;
    }
    if (T > 1 && has_la && grp == KS - 1 && tid < BC) {
        // border terms of the channel, in the order of operations of conv_epilogue.h
        // (an image of one row or column: its pixels have only the middle taps)
        const double ldw = (double)a.l_a * (double)la_dw, llw = (double)a.l_a * (double)la_lw;
        if (wide) {
            // (what the table of 25 classes is made from, behind the main loop)
#pragma unroll
            for (int t = 0; t < T; ++t) reinterpret_cast<int *>(wt_lds)[t * BC + tid] = la_sw[t];
            wt_lds[5 * BC + tid] = ldw;
            wt_lds[6 * BC + tid] = llw;
        } else {
            const bool row = a.H == 1 && a.pad > 0, column = a.W == 1 && a.pad > 0;
#pragma unroll
            for (int t = 0; t < T; ++t)
                if ((row && t / R != 1) || (column && t % R != 1)) la_sw[t] = 0;
#pragma unroll
            for (int k = 0; k < 9; ++k) {
                const int r0 = k / 3 == 1, r1 = k / 3 == 2 ? 2 : 3, c0 = k % 3 == 1, c1 = k % 3 == 2 ? 2 : 3;
                int sw = 0;
#pragma unroll
                for (int t = 0; t < T; ++t)
                    if (t / R >= r0 && t / R < r1 && t % R >= c0 && t % R < c1) sw += la_sw[t];
                const int taps = (row ? 1 : r1 - r0) * (column ? 1 : c1 - c0);
                wt_lds[k * BC + tid] = ldw * (double)sw + (double)(a.C_in * taps) * llw;
            }
        }
    }
    if (RQ && grp == KS - 1 && tid < BC) {       // (whole waves: BC is a multiple of 64)
        if (a.rq_scale == nullptr) raw.z = 1.0f;
        if (a.rq_shift == nullptr) raw.w = 0.0f;
        raw_lds[tid] = raw;
        // (RAWF below: the FP4 accumulators are used as they are, in quarter units)
        float d = chained_channel_constants(a, rq_o < a.C_out, raw.x, raw.y, raw.z, raw.w, F4 && KS == 1 ? 4.0f : 1.0f, ft_lds[tid]);
#pragma unroll
        for (int sft = 32; sft >= 1; sft >>= 1) d = __builtin_fmaxf(d, __shfl_xor(d, sft));
        if (lane == 0) te_lds[tid >> 6] = d;
    }
    lds_barrier();

    // stage i of this group works on channel block grp + i*KS.  Stages that have a
    // successor prefetch it; the last stage of a group is peeled off the loop.
    const int n_iter = (NCB + KS - 1) / KS;                  // stages of group 0
    const int n_full = (NCB - 1 - grp) / KS;                 // stages of this group with a successor
    for (int i = 0; i < n_full; ++i) {
        const int cb = grp + i * KS;
        fetch_patch(cb + KS);
        compute(std::true_type{}, patch_buf(i & 1), cb, cb + KS, patch_buf((i + 1) & 1));
        lds_barrier();
    }
    // ---- side values of the epilogue (see conv_epilogue.h for the algebra) ------
    const int top = (1 << a.bits) - 1;
    // per fragment: SA = code sums of the patch pixels under the taps (0 in the padding)
    double dsa[PF];
    float fsa[PF];          // (the same sums in binary32: exact, they stay below 2^24 wherever this is used)
    auto sum_sa = [&]() {
#pragma unroll
        for (int f = 0; f < PF; ++f) {
            int sa = 0;
#pragma unroll
            for (int t = 0; t < T; ++t) sa += pix_lds[frag_pp[f] + (t / R) * pl.PC + (t % R)];
            dsa[f] = (double)sa;
            fsa[f] = (float)sa;
        }
    };
    // Da*Dw and Da*l_w of this lane's channels of one tile: 4 groups of 4
    auto load_pq = [&](int c, double (&P)[16], double (&Q)[16]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int ol = (wc * CT + c) * 32 + 8 * q + 4 * h;   // channel inside the workgroup
#pragma unroll
            for (int j = 0; j < 4; ++j) { P[4 * q + j] = pq_lds[ol + j]; Q[4 * q + j] = pq_lds[BC + ol + j]; }
        }
    };
    // With two wave groups (two waves per SIMD, registers to spare) a wave finishes a
    // single tile; its constants and code sums are fetched before the last stage so
    // that these LDS reads run under the matrix instructions instead of after them.
    // (The tables were written before the first barrier.)
    double P0[16], Q0[16];
    const bool early_tables = KS == 2 && CT == 2;
    if (early_tables) {
        sum_sa();
        if (OUT == OUT_PLAIN) load_pq(grp, P0, Q0);
    }
    if (grp + n_full * KS < NCB) compute(std::false_type{}, patch_buf(n_full & 1), grp + n_full * KS, 0, nullptr);
    // every wave of the workgroup takes part in n_iter - 1 stage barriers
    if (KS > 1)
        for (int i = n_full; i < n_iter - 1; ++i) lds_barrier();

    // the exact integer sums (the FP4 form accumulates them in quarter units)
    v16i acc[PF][CT];
    if constexpr (!(RQ && F4 && KS == 1)) {
#pragma unroll
        for (int f = 0; f < PF; ++f)
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                if constexpr (F4) acc[f][c] = dsq_fp4_acc_to_int(macc[f][c]);
                else acc[f][c] = macc[f][c];
            }
    }

    // ---- epilogue --------------------------------------------------------------
    if (!early_tables) sum_sa();

    // The results of a 32x32 tile sit in the lanes as [pixel = lane%32][4 groups
    // of 4 channels].  They are staged through this wave's slice of the (now idle)
    // patch buffers so that each store instruction writes the 32 consecutive
    // channels (128 bytes) of 8 pixels instead of 16 bytes of 32 pixels.
    constexpr int ROWB = 128 + 16;                // staged bytes per pixel (+16: bank spread)
    constexpr int EPI_WAVE = 32 * ROWB + PF * 128;
    // chained mode, one wave group: the code-unit form reads the FP4 accumulators as
    // they are (quarter units); the integers are only formed where the exact sequence runs
    constexpr bool RAWF = RQ && F4 && KS == 1;
    lds_barrier();                              // every wave is done with the patch buffers
    if (KS == 2) {
        // each group finishes the channel tiles c with c % 2 == grp: it hands the
        // partial sums of the other tiles to its partner wave through LDS and adds
        // the partner's partial sums to its own tiles (integer adds: exact in any
        // order)
        static_assert(KS == 1 || CT % 2 == 0, "two wave groups split the channel tiles evenly");
        char *part = lds + 8 * EPI_WAVE + lane * 16;
        const int mine = (grp * 4 + wave) * (PF * (CT / 2) * 4096);
        const int theirs = ((1 - grp) * 4 + wave) * (PF * (CT / 2) * 4096);
#pragma unroll
        for (int f = 0; f < PF; ++f)
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                if ((c & 1) == grp) continue;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<v4i *>(part + mine + ((f * (CT / 2) + c / 2) * 4 + q) * 1024) =
                        (v4i){acc[f][c][4 * q], acc[f][c][4 * q + 1], acc[f][c][4 * q + 2], acc[f][c][4 * q + 3]};
            }
        lds_barrier();
#pragma unroll
        for (int f = 0; f < PF; ++f)
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                if ((c & 1) != grp) continue;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const v4i o4 = *reinterpret_cast<const v4i *>(part + theirs + ((f * (CT / 2) + c / 2) * 4 + q) * 1024);
                    acc[f][c][4 * q] += o4.x; acc[f][c][4 * q + 1] += o4.y;
                    acc[f][c][4 * q + 2] += o4.z; acc[f][c][4 * q + 3] += o4.w;
                }
            }
    }
    // border terms of the workgroup's channels, [class][channel]
    int border_at = (int)(reinterpret_cast<char *>(wt_lds) - lds);
    if (wide) {
        // Two rows of padding: pixels that lack two rows or columns of taps have classes too.  Their table takes
        // the place of the partial sums, behind the staging (25 classes do not fit beside the largest patches).
        // us, added up from the taps for every output of such a layer (which also kept the compiler from unrolling
        // the loops of OUT_GENERAL: the 256x128 tile's accumulators went through scratch memory, on every layer) ->
        // now: 64 -> 64 at 56x56 x 64 53 -> 19.3, 4 bits 72 -> 23.5, 128 -> 128 at 28x28 x 64 to NCHW 57 -> 18;
        // the 256x128 tile to NCHW, 256 -> 512 at 28x28 x 32, 46 -> 29.5.
        if (KS == 2) lds_barrier();
        border_at = 4 * KS * EPI_WAVE;
        double *wide_lds = reinterpret_cast<double *>(lds + border_at);
        // a thread forms every G-th row of classes of one channel
        constexpr int G = 256 * KS / BC;
        const int ch = (int)threadIdx.x % BC, g = __builtin_amdgcn_readfirstlane((int)threadIdx.x / BC);
        const double ldw = wt_lds[5 * BC + ch], llw = wt_lds[6 * BC + ch];
        int sw[T];
#pragma unroll
        for (int t = 0; t < T; ++t) sw[t] = reinterpret_cast<const int *>(wt_lds)[t * BC + ch];
#pragma unroll
        for (int kr = 0; kr < 5; ++kr) {
            if (kr % G != g) continue;
            const int r0 = kr == 3 ? 2 : kr == 1 || (kr == 0 && a.H == 1), r1 = kr == 4 ? 1 : kr == 2 || (kr == 0 && a.H == 1) ? 2 : 3;
            int s[3] = {0, 0, 0};                    // sums of the columns over the class's rows
#pragma unroll
            for (int t = 0; t < T; ++t) s[t % R] += t / R >= r0 && t / R < r1 ? sw[t] : 0;
#pragma unroll
            for (int kc = 0; kc < 5; ++kc) {
                const bool one = kc == 0 && a.W == 1;
                const int sum = kc == 3 ? s[2] : kc == 4 ? s[0] : s[1] + (kc == 1 || one ? 0 : s[0]) + (kc == 2 || one ? 0 : s[2]);
                const int columns = kc >= 3 || one ? 1 : kc == 0 ? 3 : 2;
                wide_lds[(kr * 5 + kc) * BC + ch] = ldw * (double)sum + (double)(a.C_in * ((r1 - r0) * columns)) * llw;
            }
        }
        lds_barrier();
    }
    // (16-byte aligned either way, which the compiler has to see to read two terms at once)
    const double *border_lds = reinterpret_cast<const double *>(lds + (border_at & ~15));
    char *stage = lds + (grp * 4 + wave) * EPI_WAVE;
    int *m_stage = reinterpret_cast<int *>(stage + 32 * ROWB);

    if (RQ) {
        // chained mode: the next layer's packed codes and pixel code sums instead
        // of the fp32 tensor (no transposition needed: a lane pair holds whole
        // 8-channel words of its pixel)
        int psum[PF];
#pragma unroll
        for (int f = 0; f < PF; ++f) psum[f] = 0;
        // (l_a = 0 here: the host sends chained layers with l_a != 0 to the split-K kernel for
        // few output tiles or the simple kernel.  Constants are fetched four channels at a time, right before
        // their use, to keep the register footprint of this path small.  Lanes of tile
        // pixels past the end compute on patch pixel 0 and are never stored; at worst
        // they send their wave through the exact sequence once more.)
        const float t_lo = a.rq_t_lo, t_hi = a.rq_t_hi;
        float near_wg = te_lds[0];
#pragma unroll
        for (int i = 1; i < BC / 64; ++i) near_wg = __builtin_fmaxf(near_wg, te_lds[i]);
        // this lane's share of the codes: a pixel's 32 channels of a tile lie in the two lanes of
        // a pair, which exchange halves so that each holds two whole words (4-bit containers) or
        // one (2-bit) of it
        const bool four = dsq_container(a.rq_bits) == 4;
        char *dst[PF];
#pragma unroll
        for (int f = 0; f < PF; ++f) {
            const size_t at = (size_t)(frag_m[f] < 0 ? 0 : frag_m[f]) * a.rq_Cp;
            dst[f] = (char *)a.rq_codes + (four ? at / 2 + 8 * h : at / 4 + 4 * h);
        }
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            if (KS == 2 && (c & 1) != grp) continue;
            const int o_tile = (ct0 + c) * 32;
            const int ol = (wc * CT + c) * 32 + 4 * h;   // this lane's first channel inside the workgroup
            // The code in code units, T = A*(ACC + rho*SA) + (B*SA + s) (see
            // chained_channel_constants): eight or nine binary32 instructions per output,
            // no binary64; the constants of four channels serve all fragments.  near[f][q]: the
            // smallest distance of a T from a half-integer among four outputs of fragment f.
            uint32_t bytes[PF][4];
            float near[PF][4];
            float4 k[2][4];
#pragma unroll
            for (int j = 0; j < 4; ++j) k[0][j] = ft_lds[ol + j];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (q < 3) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) k[(q + 1) & 1][j] = ft_lds[ol + 8 * (q + 1) + j];
                }
#pragma unroll
                for (int f = 0; f < PF; ++f) {
                    uint32_t b = 0;
                    float least = 1.0f;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float4 kj = k[q & 1][j];
                        float fa;
                        if constexpr (RAWF) fa = macc[f][c][4 * q + j];
                        else fa = (float)acc[f][c][4 * q + j];
                        const float u = __builtin_fmaf(fsa[f], kj.y, fa);
                        const float t = __builtin_fmaf(u, kj.x, __builtin_fmaf(fsa[f], kj.z, kj.w));
                        const float tc = __builtin_amdgcn_fmed3f(t, t_lo, t_hi);
                        b = __builtin_amdgcn_cvt_pk_u8_f32(tc, j, b);        // (rounds to nearest)
                        least = __builtin_fminf(least, __builtin_fabsf(__builtin_amdgcn_fractf(tc) - 0.5f));
                    }
                    bytes[f][q] = b;
                    near[f][q] = least;
                }
            }
            const int left = a.C_out - (o_tile + 4 * h);      // channels from this lane's first one on
#pragma unroll
            for (int f = 0; f < PF; ++f) {
                const float least = __builtin_fminf(__builtin_fminf(near[f][0], near[f][1]), __builtin_fminf(near[f][2], near[f][3]));
                if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(least > near_wg)) != 0, 0)) {
                    // the exact sequence: the binary32 value the plain call stores, scale,
                    // shift, ReLU and the quantizer's recipe.  (Through this wave's idle slice of
                    // the patch buffers, so that the loop needs no copy of itself per register:
                    // code that seldom runs is not in the instruction cache when it does.  Only the
                    // groups of channels that need it, as a rule one: the wave that has one is
                    // the last of its launch)
                    const int top_n = (1 << a.rq_bits) - 1;
                    const double da = (double)a.delta_a;
                    v4i *ex = reinterpret_cast<v4i *>(stage) + lane;
                    uint32_t which = 0;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        if (__builtin_amdgcn_ballot_w64(!(near[f][q] > near_wg)) == 0) continue;
                        which |= 1u << q;
                        v4i t;
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            if constexpr (RAWF) t[j] = (int)(macc[f][c][4 * q + j] * 4.0f);
                            else t[j] = acc[f][c][4 * q + j];
                        }
                        ex[64 * q] = t;
                    }
#pragma unroll 1
                    for (uint32_t todo = which; todo != 0; todo &= todo - 1) {
                        const int q = __builtin_ctz(todo);
                        const v4i t = ex[64 * q];
                        int cd[4];
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const float4 r4 = raw_lds[ol + 8 * q + j];
                            const float y = (float)__builtin_fma(da * (double)r4.x, (double)t[j], (da * (double)r4.y) * (double)fsa[f]);
                            float z = y * r4.z;
                            z = z + r4.w;
                            if (a.rq_relu) z = fmaxf(z, 0.0f);
                            cd[j] = dsq_code(z, a.rq_l, a.rq_u, a.rq_delta, top_n);
                        }
                        ex[64 * q].x = (int)dsq_bytes4(cd[0], cd[1], cd[2], cd[3]);
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (which >> q & 1) bytes[f][q] = (uint32_t)ex[64 * q].x;
                }
                if (o_tile + 32 > a.C_out) {
                    // bytes of channels >= C_out are blanked (their codes must be 0)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        bytes[f][q] &= left - 8 * q >= 4 ? 0xFFFFFFFFu : left - 8 * q <= 0 ? 0u : (1u << (8 * (left - 8 * q))) - 1u;
                }
                if (a.rq_dense) {
                    dsq_requant_store32(a, frag_m[f], o_tile, h, bytes[f], 0);
                } else {
                    // (v_permlane32_swap exchanges the upper half of its first operand with the
                    // lower half of its second: lanes 0..31 get both halves' bytes of words 0 and 1,
                    // lanes 32..63 those of words 2 and 3)
                    const auto s0 = __builtin_amdgcn_permlane32_swap(bytes[f][0], bytes[f][2], false, false);
                    const auto s1 = __builtin_amdgcn_permlane32_swap(bytes[f][1], bytes[f][3], false, false);
                    const bool here = frag_m[f] >= 0 && o_tile < a.rq_Cp;
                    if (four) {
                        const v2i w = {(int)(s0[0] | s0[1] << 4), (int)(s1[0] | s1[1] << 4)};
                        if (here) *reinterpret_cast<v2i *>(dst[f] + o_tile / 2) = w;
                    } else {
                        const uint32_t w = (s0[0] | s0[1] << 2) | (s1[0] | s1[1] << 2) << 4;
                        if (here) *reinterpret_cast<uint32_t *>(dst[f] + o_tile / 4) = w;
                    }
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) psum[f] = (int)__builtin_amdgcn_sad_u8(bytes[f][q], 0u, (uint32_t)psum[f]);
            }
        }
#pragma unroll
        for (int f = 0; f < PF; ++f)
            psum[f] += (int)__builtin_amdgcn_permlane32_swap((uint32_t)psum[f], (uint32_t)psum[f], false, false)[1];
        // The waves that share a row of pixel fragments (wave columns, wave groups)
        // hand their sums to the row's first wave through their staging slices
        // (integer adds: exact in any order) ...
        constexpr int SHARE = WC * KS;
        const bool share = SHARE > 1 && a.rq_share;      // (uniform; otherwise every wave adds its own sums)
        const bool first = !share || (wc == 0 && grp == 0);
        if (share) {
            if (!first && h == 0) {
#pragma unroll
                for (int f = 0; f < PF; ++f) m_stage[f * 32 + col] = psum[f];
            }
            lds_barrier();
            if (first && h == 0) {
#pragma unroll
                for (int g = 0; g < KS; ++g)
#pragma unroll
                    for (int c2 = 0; c2 < WC; ++c2) {
                        if (g == 0 && c2 == 0) continue;
                        const int *theirs = reinterpret_cast<const int *>(lds + (g * 4 + wp + WP * c2) * EPI_WAVE + 32 * ROWB);
#pragma unroll
                        for (int f = 0; f < PF; ++f) psum[f] += theirs[f * 32 + col];
                    }
            }
        }
        // ... which adds them to the next layer's sums with one integer atomic per
        // pixel, or stores them where the workgroup holds all channels of the layer.
        // (The hand-over costs a barrier: measured, it pays where the sums can then
        // be stored and on 1x1 layers, whose time is mostly epilogue.)
        if (h == 0 && first) {
#pragma unroll
            for (int f = 0; f < PF; ++f) {
                if (frag_m[f] < 0) continue;
                if (a.rq_store) a.rq_pix[frag_m[f]] = psum[f];
                else atomicAdd(a.rq_pix + frag_m[f], psum[f]);
            }
        }
    } else if (OUT == OUT_PLAIN) {
        if (h == 0) {
#pragma unroll
            for (int f = 0; f < PF; ++f) m_stage[f * 32 + col] = frag_m[f];
        }
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            if (KS == 2 && (c & 1) != grp) continue;
            double P[16], Q[16];
            if (KS == 2 && CT == 2) {
#pragma unroll
                for (int j = 0; j < 16; ++j) { P[j] = P0[j]; Q[j] = Q0[j]; }
            } else {
                load_pq(c, P, Q);
            }
            const int o = (ct0 + c) * 32 + (lane & 7) * 4;   // channels this lane stores
#pragma unroll
            for (int f = 0; f < PF; ++f) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    double v[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        v[j] = __builtin_fma(P[4 * q + j], (double)acc[f][c][4 * q + j], Q[4 * q + j] * dsa[f]);
                    *reinterpret_cast<float4 *>(stage + col * ROWB + (8 * q + 4 * h) * 4) =
                        make_float4((float)v[0], (float)v[1], (float)v[2], (float)v[3]);
                }
                // (LDS operations of one wave execute in order: no barrier needed)
                float4 rv[4];
                int rm[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int p = k * 8 + (lane >> 3);
                    rv[k] = *reinterpret_cast<const float4 *>(stage + p * ROWB + (lane & 7) * 16);
                    rm[k] = m_stage[f * 32 + p];
                }
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (rm[k] >= 0 && o < a.C_out)
                    {
                        // non-temporal: the output is not read again by this kernel, and
                        // streaming it out as it is produced leaves less for the write-back
                        // at the end of the kernel (measured 5-25 % off the kernel time of
                        // every layer class; a consumer that runs right after finds less of
                        // the tensor in the last-level cache, which costs it about as much)
                        typedef float v4f __attribute__((ext_vector_type(4)));
                        const v4f t = {rv[k].x, rv[k].y, rv[k].z, rv[k].w};
                        __builtin_nontemporal_store(t, reinterpret_cast<v4f *>(a.out + (size_t)rm[k] * a.C_out + o));
                    }
            }
        }
    } else if (OUT == OUT_ROWS) {
        // The values of OUT_PLAIN plus, for l_a != 0, the terms of conv_epilogue.h that depend on
        // which taps lie inside the image, in its order of operations (the same bits).  A lane
        // holds one channel of 16 pixels, so that a channel's binary64 constants stay in registers:
        // with the pixel in the lane they come from LDS for every output, which keeps the LDS busy
        // for 0.6 of the time on 1x1 layers.  The pixels' code sums and places come from LDS, for all
        // channel tiles at once; a store writes 128 consecutive bytes of two pixels.  Channel tiles
        // past C_out are left out.
        double *sa_stage = reinterpret_cast<double *>(stage);                       // [fragment][pixel]
        int *at_stage = reinterpret_cast<int *>(stage + PF * 256), *cls_stage = at_stage + PF * 32;
        if (h == 0) {
#pragma unroll
            for (int f = 0; f < PF; ++f) {
                sa_stage[f * 32 + col] = dsa[f];
                at_stage[f * 32 + col] = frag_m[f] < 0 ? -1 : frag_m[f] * a.C_out;   // (an element index: below 2^31)
                cls_stage[f * 32 + col] = frag_cls[f] * BC;
            }
        }
        double P[CT], Q[CT], W[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const int ol = (wc * CT + c) * 32 + col;
            P[c] = pq_lds[ol];
            Q[c] = pq_lds[BC + ol];
            W[c] = has_la ? border_lds[ol] : 0.0;
        }
#pragma unroll
        for (int f = 0; f < PF; ++f) {
            // (LDS operations of one wave execute in order: no barrier needed)
            const bool border = T > 1 && has_la && __builtin_amdgcn_ballot_w64(frag_cls[f] != 0) != 0;
            const bool all = __builtin_amdgcn_ballot_w64(frag_m[f] < 0) == 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                double sa[4];
                int at[4], cls[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    sa[j] = sa_stage[f * 32 + 8 * q + 4 * h + j];
                    at[j] = at_stage[f * 32 + 8 * q + 4 * h + j];
                    cls[j] = border ? cls_stage[f * 32 + 8 * q + 4 * h + j] : 0;
                }
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    if (KS == 2 && (c & 1) != grp) continue;
                    const int o_tile = (ct0 + c) * 32, o = o_tile + col, ol = (wc * CT + c) * 32 + col;
                    if (o_tile >= a.C_out) continue;
                    float res[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        double v = __builtin_fma(P[c], (double)acc[f][c][4 * q + j], Q[c] * sa[j]);
                        if (has_la) v += border ? border_lds[cls[j] + ol] : W[c];
                        res[j] = (float)v;
                    }
                    if (all && o_tile + 32 <= a.C_out) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) __builtin_nontemporal_store(res[j], a.out + (size_t)(uint32_t)at[j] + o);
                    } else {
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            if (at[j] >= 0 && o < a.C_out) a.out[(size_t)(uint32_t)at[j] + o] = res[j];
                    }
                }
            }
        }
    } else {
        // The values of OUT_PLAIN plus, for l_a != 0, the terms of conv_epilogue.h that depend on
        // which taps lie inside the image, from the table of its class, in its order of
        // operations (the same bits).  NCHW: the accumulator layout already has 32
        // consecutive pixels of a channel in 32 lanes, so each store writes two runs of 128
        // bytes.  NHWC (with raw accumulators): staged like OUT_PLAIN, in single floats where C_out
        // is not a multiple of 4.  Bound by the store of the tensor; 128 -> 256 stride 2 at 28x28 x 64
        // to NCHW 14 us; with l_a != 0 (tap sums added up for every pixel at a border -> now): 64 -> 64
        // at 32x32 x 1 9.2 -> 6.5, 64 -> 64 at 56x56 x 64 23.4 -> 19.0, 256 -> 256 at 14x14 x 64 16.5 -> 13.8.
        if (h == 0) {
#pragma unroll
            for (int f = 0; f < PF; ++f) m_stage[f * 32 + col] = frag_m[f];
        }
        const int plane = a.Ho * a.Wo;
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            if (KS == 2 && (c & 1) != grp) continue;
            const int o_tile = (ct0 + c) * 32;
            const int ol = (wc * CT + c) * 32 + 4 * h;     // this lane's first channel inside the workgroup
#pragma unroll
            for (int f = 0; f < PF; ++f) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int o0 = o_tile + 8 * q + 4 * h;
                    double v[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        v[j] = __builtin_fma(pq_lds[ol + 8 * q + j], (double)acc[f][c][4 * q + j],
                                             pq_lds[BC + ol + 8 * q + j] * dsa[f]);
                    if (has_la) {
                        double w[4];
#pragma unroll
                        for (int j = 0; j < 4; ++j) w[j] = border_lds[frag_cls[f] * BC + ol + 8 * q + j];
#pragma unroll
                        for (int j = 0; j < 4; ++j) v[j] += w[j];
                    }
                    if (a.out_nchw) {
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            if (frag_m[f] >= 0 && o0 + j < a.C_out)
                                a.out[(size_t)frag_base[f] + (size_t)(o0 + j) * plane] = (float)v[j];
                    } else {
                        *reinterpret_cast<float4 *>(stage + col * ROWB + (8 * q + 4 * h) * 4) =
                            make_float4((float)v[0], (float)v[1], (float)v[2], (float)v[3]);
                    }
                    if (a.acc != nullptr && frag_m[f] >= 0) {
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            if (o0 + j < a.C_out)
                                a.acc[a.out_nchw ? (size_t)frag_base[f] + (size_t)(o0 + j) * plane
                                                 : (size_t)frag_m[f] * a.C_out + o0 + j] = acc[f][c][4 * q + j];
                    }
                }
                if (a.out_nchw) continue;
                // (LDS operations of one wave execute in order: no barrier needed)
                if ((a.C_out & 3) == 0) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int p = k * 8 + (lane >> 3), o = o_tile + (lane & 7) * 4;
                        typedef float v4f __attribute__((ext_vector_type(4)));
                        const v4f t = *reinterpret_cast<const v4f *>(stage + p * ROWB + (lane & 7) * 16);
                        const int rm = m_stage[f * 32 + p];
                        if (rm >= 0 && o < a.C_out)
                            __builtin_nontemporal_store(t, reinterpret_cast<v4f *>(a.out + (size_t)rm * a.C_out + o));
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < 16; ++k) {
                        const int p = k * 2 + h, o = o_tile + col;
                        const float t = *reinterpret_cast<const float *>(stage + p * ROWB + col * 4);
                        const int rm = m_stage[f * 32 + p];
                        if (rm >= 0 && o < a.C_out) a.out[(size_t)rm * a.C_out + o] = t;
                    }
                }
            }
        }
    }
}

// ---- host side ---------------------------------------------------------------

// tables behind the buffers: Da*Dw, Da*l_w (binary64; chained mode: Dw, l_w, scale, shift), the
// patch pixels' code sums; then the chained mode's per-channel constants of the code-unit
// form, or the general results' tables for l_a != 0
constexpr int border_table_bytes(int R, int BC) { return (R > 1 ? 9 : 1) * BC * 8; }

inline int plan_lds_bytes(const PatchPlan &p, int BC, const DsqConvArgs &a)
{
    const int tables = (p.aux_off + 2 * BC * 8 + p.PR * p.PC * 4 + 15) & ~15;
    const int chained = BC * 16 + 16;
    return tables + (a.rq ? chained : a.l_a != 0.0f ? border_table_bytes(a.R, BC) : 0);
}

// What a plan is held against its limit with: the same for a layer with l_a != 0 as for one
// with l_a = 0 (with some room for further tables counted always), so that which layers
// and forced tiles the kernel takes does not depend on l_a.
inline int plan_limit_bytes(const PatchPlan &p, int BC, const DsqConvArgs &a)
{
    return ((p.aux_off + 2 * BC * 8 + p.PR * p.PC * 4 + 15) & ~15) + 2 * BC * 4 + 16 * 8 + (a.rq ? BC * 16 + 16 : 0);
}

template <int CONT, int R, int WP, int WC, int PF, int CT, int UPT, int WD, int OCC, int KS, int OUT>
hipError_t launch_kernel(const DsqConvArgs &a, const PatchPlan &pl, hipStream_t stream)
{
    auto kern = conv_patch_kernel<CONT, R, WP, WC, PF, CT, UPT, WD, OCC, KS, OUT>;
    const int BC = 32 * CT * WC;
    const size_t lds = (size_t)plan_lds_bytes(pl, BC, a);      // pl.aux_off already accounts for KS
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    // chained mode, layer wider than the tile: the workgroups add to the next
    // layer's pixel sums, which a fill kernel clears first (unless the caller did)
    if (OUT == OUT_CODES && !a.rq_store && !a.rq_zeroed) {
        const hipError_t e = dsq_launch_fill_zero(a.rq_pix, (size_t)a.N * a.Ho * a.Wo, stream);
        if (e != hipSuccess) return e;
    }
    PatchPlan p2 = pl;
    p2.tiles_c = (a.C_out + BC - 1) / BC;
    p2.mg_tiles_c = dsq_division_constant(p2.tiles_c);
    p2.total_blocks = pl.tiles_w * pl.row_tiles * p2.tiles_c;
    p2.xcd_chunk = (p2.total_blocks + 7) / 8;
    kern<<<dim3(8 * p2.xcd_chunk), 256 * KS, lds, stream>>>(a, p2);
    return hipGetLastError();
}

// Tile shapes (pixels x channels per workgroup; per wave PF x CT MFMA tiles):
//   small  128 x  64   waves 4x1, 1 x 2 tiles each  (few pixels: fill the chip)
//   medium 128 x 128   waves 2x2, 2 x 2
//   large  256 x 128   waves 2x2, 4 x 2
//   tall   256 x  64   waves 4x1, 2 x 2  (layers with at most 64 output channels)
template <int CONT, int R, int WP, int WC, int PF, int CT, int UPT, int WD, int OCC, int KS = 1, bool CHAINED = true>
hipError_t launch_cfg(const DsqConvArgs &a, const PatchPlan &pl, hipStream_t stream)
{
    const int out = output_mode(a, 32 * CT * WC);
    if constexpr (CHAINED)
        if (out == OUT_CODES) return launch_kernel<CONT, R, WP, WC, PF, CT, UPT, WD, OCC, KS, OUT_CODES>(a, pl, stream);
    if (out == OUT_GENERAL) return launch_kernel<CONT, R, WP, WC, PF, CT, UPT, WD, OCC, KS, OUT_GENERAL>(a, pl, stream);
    if (out == OUT_ROWS) return launch_kernel<CONT, R, WP, WC, PF, CT, UPT, WD, OCC, KS, OUT_ROWS>(a, pl, stream);
    return launch_kernel<CONT, R, WP, WC, PF, CT, UPT, WD, OCC, KS, OUT_PLAIN>(a, pl, stream);
}

enum { TILE_SMALL = 0, TILE_MEDIUM = 1, TILE_LARGE = 2, TILE_TALL = 3 };

// All variants of one (container, filter size) pair: tile, wave groups, and the
// number of 16-byte fetch units per thread (instantiated 2, 4, 8, 12).
// (The 128x64 tile with two fetch units per thread runs four waves per SIMD: layers of
// 784 k tiles, the 56x56 and 112x112 images, leave a nearly empty last round on 768
// resident workgroups; measured 5-8 % off such layers, 8-15 % off their chained call,
// no change elsewhere.  With eight units and more, the strided layers, three waves per SIMD cost 3x3 layers up to 28
// spilled registers.  A layer with a single channel block has one patch buffer, of which three fit a compute unit, and needs
// the third workgroup (us, two / three waves: 64 -> 64 stride 2 at 112x112 x 64 4 bits 26.3 / 23.1, chained 25.5 / 21.1,
// to NCHW 30.9 / 25.7); the two buffers of deeper layers, of more than 512 pixels each at 4 bits and 1024 at 2, leave room for one, and
// two waves do without the spills (256 -> 24 stride 2 at 112x112 x 16 with l_a != 0 27.1 / 28.5, 496 -> 80 at 85x85 x 5 with
// l_a != 0 to NCHW 61.9 / 64.2).)
template <int CONT, int RR>
hipError_t dispatch_variant(const DsqConvArgs &a, const PatchPlan &pl, int which, int ks, int need, hipStream_t stream)
{
#define DSQ_TILE(CONT, RR, UPT)                                                                \
    do {                                                                                       \
        if (which == TILE_LARGE) {                                                             \
            return launch_cfg<CONT, RR, 2, 2, 4, 2, UPT, (RR == 3 ? 3 : 1), 2, 1, CONT == 2>(a, pl, stream); \
        }                                                                                      \
        if (which == TILE_MEDIUM && ks == 2) return launch_cfg<CONT, RR, 2, 2, 2, 2, UPT, (RR == 3 ? 3 : 1), 2, 2>(a, pl, stream); \
        if (which == TILE_MEDIUM) return launch_cfg<CONT, RR, 2, 2, 2, 2, UPT, (RR == 3 ? 3 : 1), 3>(a, pl, stream); \
        if (which == TILE_TALL) return launch_cfg<CONT, RR, 4, 1, 2, 2, UPT, (RR == 3 ? 3 : 1), 3>(a, pl, stream); \
        if (ks == 2) return launch_cfg<CONT, RR, 4, 1, 1, 2, UPT, (RR == 3 ? 3 : 1), 2, 2>(a, pl, stream); \
        if constexpr (RR == 3 && UPT >= 8) \
            if (a.Cp > 64) return launch_cfg<CONT, RR, 4, 1, 1, 2, UPT, 3, 2>(a, pl, stream); \
        return launch_cfg<CONT, RR, 4, 1, 1, 2, UPT, (RR == 3 ? 3 : 1), (UPT == 2 ? 4 : 3)>(a, pl, stream); \
    } while (0)
#define DSQ_GO(CONT, RR)                                                                       \
    do {                                                                                       \
        if (need <= 2) DSQ_TILE(CONT, RR, 2);                                                  \
        if (need <= 4) DSQ_TILE(CONT, RR, 4);                                                  \
        if (need <= 8) DSQ_TILE(CONT, RR, 8);                                                  \
        DSQ_TILE(CONT, RR, 12);                                                                \
    } while (0)
    DSQ_GO(CONT, RR);
#undef DSQ_TILE
#undef DSQ_GO
    return hipErrorInvalidValue;
}

}  // namespace

// One translation unit per (container, filter size) pair, so that they compile side by side.
hipError_t dsq_conv_patch_c4r3(const DsqConvArgs &a, const PatchPlan &pl, int which, int ks, int need, hipStream_t stream);
hipError_t dsq_conv_patch_c4r1(const DsqConvArgs &a, const PatchPlan &pl, int which, int ks, int need, hipStream_t stream);
hipError_t dsq_conv_patch_c2r3(const DsqConvArgs &a, const PatchPlan &pl, int which, int ks, int need, hipStream_t stream);
hipError_t dsq_conv_patch_c2r1(const DsqConvArgs &a, const PatchPlan &pl, int which, int ks, int need, hipStream_t stream);
hipError_t dsq_conv_patch_c3r3(const DsqConvArgs &a, const PatchPlan &pl, int which, int ks, int need, hipStream_t stream);
hipError_t dsq_conv_patch_c3r1(const DsqConvArgs &a, const PatchPlan &pl, int which, int ks, int need, hipStream_t stream);
