// dsq_conv2d_wq: a layer whose weights are quantized and whose activations are not
// (the "b/32" rows of the paper's Tables 3, 6 and 7: b-bit weights, 32-bit
// activations).  Algorithm 1 steps 4 and 5 with a_hat = a: the binary32 activations
// are convolved with the weight levels l_w + Dw*code.
//
// The inner product runs on the bf16 matrix instruction (v_mfma_f32_32x32x16_bf16,
// 16 times the rate of the binary32 one) on exact operands:
//   - an activation is the sum of three bf16 numbers of 8 significant bits each
//     (its 24 bits cut in three; every step of the split is exact),
//   - a level is Dw*(code + zq) + lr, zq = l_w/Dw rounded so that code + zq is a
//     bf16 number for every code, lr = l_w - Dw*zq, rounded once (0 for the symmetric
//     ranges of 1-bit weights; at most Dw/128 at 2 bits and Dw/32 at 4 bits where the range
//     holds 0, more where |l_w| is larger than Dw's multiples: Dw/8 at l_w = 30*Dw; l_w
//     itself, with zq = 0, from |l_w| = 256*Dw on),
// so that out = Dw * sum (code + zq)*(x2 + x1 + x0) + lr * sum x.  Products of two
// such terms have at most 16 bits and are exact; the sums are binary32.  Three matrix
// instructions of 32 clk for 16 channels against eight of 64 clk.  Sums of centred
// levels (and not of the codes themselves) keep the partial sums as small as those of
// the levels.  The three terms of a number reach 23 binary places below it, past the
// smallest bf16 number where |x| < 2^-110: the split is made of x * 2^54 (exact, as every
// non-zero |x| is a multiple of 2^-149), whose terms and products are all normal numbers,
// and Dw is scaled back.  A tile that holds an |x| of 2^46 or more (infinities and NaN
// among them), or a step that cannot be scaled back exactly, is computed with the
// binary32 matrix instruction from the levels themselves.
//
// A workgroup owns BP output pixels of a strip of TW columns (pixels are numbered row
// by row through the batch) and BC output channels.  Per stage of KC input channels
// the input patch under its taps is read once, split, and kept in LDS (as three bf16
// planes per pixel); the R*R taps read shifted windows of it.  Weight codes go from
// global memory to registers, all of a stage's in flight while the patch is staged.
// Bound by staging between the matrix instructions (128 -> 128 3x3 at 28x28 x 64, clocks of a
// wave: set-up 4700, staging and its barriers 22000, multiplication 40000, of which 28000 are the
// matrix instruction's, results 8200) and by 392 tiles on 256 compute units: 188 us on the binary32
// instruction, 49 with levels formed one by one and a sum of x for every layer, 45 now
// (330 TFLOP/s) with the tensor in the last-level cache.
#include "dsq_device.h"
#include "dsq_kernels.h"
#include "wq_plan.h"

namespace {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr float kUp = 0x1p54f, kDown = 0x1p-54f;                     // scale of the split activations
constexpr uint32_t kMostBits = 0x71800000u;                          // 2^100: |x| = 2^46

// The wave's PF x CT tiles with the binary32 matrix instruction: the levels themselves
// (l_w + Dw*code, rounded once) times the activations, both straight from global memory, in
// steps of 8 channels of a tap and lane half (every KW-th one, from kw on).  A step's loads are in flight
// while the one before is multiplied, and its fragments are shared by the wave's tiles.  A lane
// belongs to pixel (py, px) of image n of each fragment (valid: there is one).
// Bound by the matrix instruction (64 clk for 2 channels) and by rounds of workgroups.  An
// infinity in every tile, against one wave per 32x32 tile with its loads waited for (us):
// 128->128 3x3 at 28x28 x 64 188 -> 182, 64->64 at 56x56 x 64 240 -> 194, 512->512 at 7x7 x 1
// 141 -> 66, 24->144 1x1 at 56x56 x 64 88 -> 73, 4096->4096 x 64 153 -> 96; 64->128 stride 2
// at 56x56 x 64 101 -> 119 (two stages, one of them split in vain).
template <int R, int KW, int PF, int CT, bool VEC>
__device__ __forceinline__ void wq_exact_tiles(const DsqConvArgs &a, const float *__restrict__ x, int x_nchw, int lane, int kw, int ct0,
                                               const int (&m)[PF], const int (&n)[PF], const int (&py)[PF], const int (&px)[PF],
                                               v16f (&acc)[PF][CT])
{
    constexpr int T = R * R;
    const int col = lane & 31, h = lane >> 5;
    const int NCB = a.Cp / 64;
    // a lane half has 32 channels of a block in four words, 0..7 / 16..23 of it in the first: the last block's
    // words that start past C_in are left out
    const int rest = a.C_in - 64 * (NCB - 1), words = 1 + (rest > 8) + (rest > 32) + (rest > 40);
    const int steps = ((NCB - 1) * 4 + words) * T;
    const int live = (a.C_out + 31) / 32 - ct0;           // tiles with channels
    const int cs = x_nchw ? a.H * a.W : 1, ps = x_nchw ? 1 : a.C_in;      // strides of channels and of pixels
    int at[PF], taps[PF];                                 // of the pixel's first tap; bit t: tap t lies inside the image
#pragma unroll
    for (int f = 0; f < PF; ++f) {
        const int iy = py[f] * a.stride - a.pad, ix = px[f] * a.stride - a.pad;
        at[f] = x_nchw ? (n[f] * a.C_in * a.H + iy) * a.W + ix : ((n[f] * a.H + iy) * a.W + ix) * a.C_in;
        taps[f] = 0;
#pragma unroll
        for (int t = 0; t < T; ++t)
            if (m[f] >= 0 && (unsigned)(iy + t / R) < (unsigned)a.H && (unsigned)(ix + t % R) < (unsigned)a.W) taps[f] |= 1 << t;
    }
    float dw[CT], lw[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) { dw[c] = a.delta_w[(ct0 + c) * 32 + col]; lw[c] = a.l_w[(ct0 + c) * 32 + col]; }
#pragma unroll
    for (int f = 0; f < PF; ++f)
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[f][c][r] = 0.f;

    struct Step { v4f v[PF][2]; uint32_t w[CT]; bool inside[PF]; int c0; };
    auto load = [&](int s, Step &st) {
        const int t = s % T, w = s / T % 4, cb = s / T / 4;
        st.c0 = 64 * cb + 32 * (w >> 1) + 16 * h + 8 * (w & 1);
#pragma unroll
        for (int c = 0; c < CT; ++c)
            st.w[c] = ((const uint32_t *)a.wq)[((((size_t)(ct0 + c) * NCB + cb) * T + t) * 64 + lane) * 4 + w];
#pragma unroll
        for (int f = 0; f < PF; ++f) {
            st.inside[f] = taps[f] >> t & 1;
            // (branch-free: what does not exist reads the tensor's first values and is blanked below)
            const float *p = x + (st.inside[f] ? at[f] + (t / R * a.W + t % R) * ps : 0);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int c = st.c0 + 4 * q;
                if constexpr (VEC) st.v[f][q] = *reinterpret_cast<const v4f *>(p + (c < a.C_in ? c : 0));
                else
#pragma unroll
                    for (int j = 0; j < 4; ++j) st.v[f][q][j] = p[c + j < a.C_in ? (size_t)(c + j) * cs : 0];
            }
        }
    };
    auto multiply = [&](const Step &st) {
        float v[PF][8];                                   // padding and channels >= C_in: the real number 0
#pragma unroll
        for (int f = 0; f < PF; ++f)
#pragma unroll
            for (int j = 0; j < 8; ++j)
                v[f][j] = st.inside[f] && st.c0 + (VEC ? j & 4 : j) < a.C_in ? st.v[f][j >> 2][j & 3] : 0.f;
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            if (c >= live) continue;
            uint32_t b[2];
            dsq_unpack4(st.w[c], b[0], b[1]);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float level = __builtin_fmaf(dw[c], (float)((b[j >> 2] >> (8 * (j & 3))) & 0xFFu), lw[c]);
#pragma unroll
                for (int f = 0; f < PF; ++f) acc[f][c] = __builtin_amdgcn_mfma_f32_32x32x2f32(level, v[f][j], acc[f][c], 0, 0, 0);
            }
        }
    };
    Step even, odd;
    // (loads without a branch, the last step's again past the end: the compiler then knows how many
    // are in flight behind the one it waits for)
    load(min(kw, steps - 1), even);
    for (int s = kw; s < steps; s += 2 * KW) {
        load(min(s + KW, steps - 1), odd);
        multiply(even);
        load(min(s + 2 * KW, steps - 1), even);
        if (s + KW < steps) multiply(odd);
    }
}

// zq of a channel: l/d on the grid on which every code + zq, code <= top, has 8
// significant bits; 0 where no such grid holds the integers (|l| >> d, or d = 0).
__device__ __forceinline__ float centre_of(float l, float d, int top)
{
    const double z = (double)l / (double)d;
    const double m = __builtin_fmax(__builtin_fabs(z), __builtin_fabs(z + top));
    if (!(m < 256.0)) return 0.0f;
    const int e = max(__builtin_amdgcn_frexp_exp(m), 0);  // 2^(e-1) <= m < 2^e (m >= top/2)
    return (float)__builtin_amdgcn_ldexp(__builtin_rint(__builtin_amdgcn_ldexp(z, 8 - e)), e - 8);      // grid 2^(e-8)
}

// WP x WC waves of PF x CT 32x32 tiles; KW > 1: the waves share one such block and
// take every KW-th 16-channel step of K (layers that yield few blocks).
// VEC: NHWC activations with whole float4s (C_in a multiple of 4).
// LUT: codes of at most 3 bits, whose centred levels a lane keeps as two tables of eight bytes
// (low and high halves of the bf16 numbers): v_perm_b32 looks four codes up at once, 11 vector
// instructions for eight levels where forming them takes 28.
template <int R, int WP, int WC, int KW, int PF, int CT, int OCC, bool VEC, bool LUT>
__global__ __launch_bounds__(256, OCC) void conv_wq_kernel(DsqConvArgs a, const float *__restrict__ x, int x_nchw, int top, WqPlan pl)
{
    constexpr int T = R * R;
    constexpr int KC = kc_of(R), G = KC / 8, STEPS = T * KC / 16, NS = (STEPS + KW - 1) / KW;
    constexpr int PIXB = pixel_bytes(R);
    constexpr int BP = 32 * PF * WP, BC = 32 * CT * WC;
    static_assert(WP * WC * KW == 4 && (KW == 1 || KW == 4) && BC <= 256, "four waves per workgroup");
    extern __shared__ __attribute__((aligned(16))) char lds[];
    float *sx_lds = reinterpret_cast<float *>(lds + tables_at(R, KW, PF * CT, pl.npx));
    int *addr_lds = reinterpret_cast<int *>(sx_lds + G * pl.npx);
    float *zq_lds = reinterpret_cast<float *>(addr_lds + pl.npx);
    float *dw_lds = zq_lds + BC, *lr_lds = dw_lds + BC;
    int *whole_lds = reinterpret_cast<int *>(lr_lds + BC);

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, h = lane >> 5;
    const int kw = KW == 1 ? 0 : wave, wp = KW == 1 ? wave % WP : 0, wc = KW == 1 ? wave / WP : 0;

    // every XCD (workgroups are dealt to them in turn) gets a contiguous range of tiles
    const int logical = ((int)blockIdx.x & 7) * pl.xcd_chunk + ((int)blockIdx.x >> 3);
    if (logical >= pl.total_blocks) return;
    int blk_c, tile_w, tc0, oh0;
    const int blk_p = dsq_idiv(logical, pl.tiles_c, pl.mg_tiles_c, blk_c);
    const int t0 = dsq_idiv(blk_p, pl.tiles_w, pl.mg_tiles_w, tile_w) * BP;
    const int ow0 = tile_w * pl.TW, NHo = a.N * a.Ho;
    const int gr0 = dsq_idiv(t0, pl.TW, pl.mg_TW, tc0);
    const int n0 = dsq_idiv(gr0, a.Ho, pl.mg_Ho, oh0);
    const int v0 = n0 * pl.Hp + oh0 * a.stride;           // first padded input row of the patch
    const int ct0 = blk_c * (BC / 32) + wc * CT;
    const int NCB = a.Cp / 64;

    // ---- tables: where the patch pixels are, and the channels' constants ---------
    static_assert(BC <= 128, "two flags");
    if (lane == 0 && wave < 2) whole_lds[1 + wave] = 0;   // (this wave's own, read behind the barrier)
    for (int p = tid; p < pl.npx; p += 256) {
        int n, ih, iw;
        bool ok;
        if (R == 1) {
            int tc, oh;
            const int gr = dsq_idiv(t0 + p, pl.TW, pl.mg_TW, tc);
            n = dsq_idiv(gr, a.Ho, pl.mg_Ho, oh);
            ok = gr < NHo;
            ih = oh * a.stride; iw = tc * a.stride;
        } else {
            int pcol;
            const int prow = dsq_idiv(p, pl.PC, pl.mg_PC, pcol);
            n = dsq_idiv(v0 + prow, pl.Hp, pl.mg_Hp, ih);
            ih -= a.pad; iw = ow0 * a.stride + pcol - a.pad;
            ok = n < a.N && (unsigned)ih < (unsigned)a.H && (unsigned)iw < (unsigned)a.W;
        }
        addr_lds[p] = !ok ? -1 : x_nchw ? (n * a.C_in * a.H + ih) * a.W + iw : ((n * a.H + ih) * a.W + iw) * a.C_in;
    }
    bool unscalable = false;                              // Dw * 2^-54 is not exact (or Dw infinite)
    if (tid < BC) {
        const float d = a.delta_w[blk_c * BC + tid], l = a.l_w[blk_c * BC + tid];      // (Cop covers them)
        const float zq = centre_of(l, d, top);
        zq_lds[tid] = zq;
        dw_lds[tid] = d * kDown;
        unscalable = __builtin_fabsf(d) == __builtin_inff() || (d != 0.0f && __builtin_fabsf(d) < 0x1p-72f);
        const float lr = (float)((double)l - (double)d * (double)zq);
        lr_lds[tid] = lr;
        // (a NaN counts)
        if (__builtin_amdgcn_ballot_w64(!(lr == 0.0f)) != 0 && lane == 0) whole_lds[1 + wave] = 1;
    }
    if (tid == 0) *whole_lds = 0;
    __syncthreads();
    // sums of x are taken where a channel's levels have a remainder off the grid
    const bool sums = __builtin_amdgcn_readfirstlane(whole_lds[1] | whole_lds[2]) != 0;

    // ---- the lane's pixels and weight rows ----------------------------------------
    int frag_off[PF], frag_pp[PF], frag_m[PF], frag_n[PF], frag_y[PF], frag_x[PF];
#pragma unroll
    for (int f = 0; f < PF; ++f) {
        const int p = (wp * PF + f) * 32 + col;
        int tc, oh;
        const int gr = dsq_idiv(t0 + p, pl.TW, pl.mg_TW, tc);
        const int n = dsq_idiv(gr, a.Ho, pl.mg_Ho, oh);
        const bool ok = gr < NHo && ow0 + tc < a.Wo;
        frag_m[f] = ok ? gr * a.Wo + ow0 + tc : -1;
        frag_n[f] = n; frag_y[f] = oh; frag_x[f] = ow0 + tc;
        // (pixels past the end multiply patch pixel 0 and are never stored)
        frag_pp[f] = R == 1 ? p : ok ? (n * pl.Hp + oh * a.stride - v0) * pl.PC + tc * a.stride : 0;
        frag_off[f] = frag_pp[f] * PIXB + 32 * h;
    }
    float zq[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) zq[c] = zq_lds[(wc * CT + c) * 32 + col];
    uint32_t tab[CT][4];                                  // low bytes of codes 0..3, 4..7, high bytes of the same
    if constexpr (LUT) {
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                uint32_t e[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) e[j] = __float_as_uint((float)(4 * i + j) + zq[c]);
                const uint32_t p01 = __builtin_amdgcn_perm(e[1], e[0], 0x07030602u), p23 = __builtin_amdgcn_perm(e[3], e[2], 0x07030602u);
                tab[c][i] = __builtin_amdgcn_perm(p23, p01, 0x05040100u);
                tab[c][2 + i] = __builtin_amdgcn_perm(p23, p01, 0x07060302u);
            }
    }

    v16f acc[PF][CT];
#pragma unroll
    for (int f = 0; f < PF; ++f)
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[f][c][r] = 0.f;

    // ---- staging ---------------------------------------------------------------------
    const int HW = a.H * a.W;
    uint32_t max_bits = unscalable ? kMostBits : 0;       // largest |x| * 2^54, as its bits
    uint32_t seen = 0;                                    // all weight words or'ed together
    auto put = [&](int px, int g, bool first, const float (&v)[8]) {
        uint32_t hi[8], mid[8], lo[8];
        float s = 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float z = v[j] * kUp;
            const uint32_t b = __float_as_uint(z);
            max_bits = max(max_bits, b & 0x7FFFFFFFu);
            hi[j] = b & 0xFFFF0000u;
            const float r1 = z - __uint_as_float(hi[j]);
            mid[j] = __float_as_uint(r1) & 0xFFFF0000u;
            lo[j] = __float_as_uint(r1 - __uint_as_float(mid[j]));
        }
        v4i w[3];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            w[0][j] = (int)__builtin_amdgcn_perm(hi[2 * j + 1], hi[2 * j], 0x07060302u);
            w[1][j] = (int)__builtin_amdgcn_perm(mid[2 * j + 1], mid[2 * j], 0x07060302u);
            w[2][j] = (int)__builtin_amdgcn_perm(lo[2 * j + 1], lo[2 * j], 0x07060302u);
        }
#pragma unroll
        for (int p = 0; p < 3; ++p) *reinterpret_cast<v4i *>(lds + px * PIXB + p * KC * 2 + g * 16) = w[p];
        if (sums) {
#pragma unroll
            for (int j = 0; j < 8; ++j) s += v[j];
            sx_lds[g * pl.npx + px] = first ? s : sx_lds[g * pl.npx + px] + s;
        }
    };
    // Unit k of a thread: one patch pixel, 8 channels.  NHWC with whole float4s: a thread keeps
    // its channels and the G groups of a pixel sit in neighbouring lanes; otherwise (NCHW, odd
    // C_in) a wave keeps its channels and its lanes run along the pixels.
    const int n_units = VEC ? (pl.npx + 256 / G - 1) / (256 / G) : (pl.npx + 63) / 64 * (G / 4);
    auto unit_px = [&](int k) { return VEC ? tid / G + k * (256 / G) : lane + k / (G / 4) * 64; };
    auto unit_g = [&](int k) { return VEC ? tid % G : wave + 4 * (k % (G / 4)); };
    // (branch-free: what does not exist reads the tensor's first values and is blanked below)
    auto load_unit = [&](int k, int st, float (&v)[8]) {
        const int q = unit_px(k), c0 = st * KC + 8 * unit_g(k);
        const int ad = q < pl.npx ? addr_lds[q] : -1;
        const float *p = x + (ad >= 0 ? ad : 0);
        if constexpr (VEC) {
            const v4f lo4 = *reinterpret_cast<const v4f *>(p + (c0 < a.C_in ? c0 : 0));
            const v4f hi4 = *reinterpret_cast<const v4f *>(p + (c0 + 4 < a.C_in ? c0 + 4 : 0));
#pragma unroll
            for (int j = 0; j < 4; ++j) { v[j] = lo4[j]; v[4 + j] = hi4[j]; }
        } else {
            const int cs = x_nchw ? HW : 1;
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = p[c0 + j < a.C_in ? (size_t)(c0 + j) * cs : 0];
        }
    };
    auto put_unit = [&](int k, int st, const float (&raw)[8]) {
        const int q = unit_px(k), g = unit_g(k), c0 = st * KC + 8 * g;
        if (q >= pl.npx) return;
        const bool on = addr_lds[q] >= 0;
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = on && c0 + j < a.C_in ? raw[j] : 0.f;
        put(q, g, st == 0, v);
    };
    const int stages = (a.C_in + KC - 1) / KC;
    int whole = 0;
    for (int st = 0; st < stages; ++st) {
        // the stage's weight words of this wave: step s = tap, 16-channel slice
        const int cb = st * KC / 64;
        uint32_t wreg[NS][CT];
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            int s = kw + KW * j;
            if (KW > 1 && s >= STEPS) s = STEPS - 1;
            const int t = s / (KC / 16), sl = s % (KC / 16) + (KC == 32 ? 2 * (st & 1) : 0);
#pragma unroll
            for (int c = 0; c < CT; ++c)
                wreg[j][c] = ((const uint32_t *)a.wq)[((((size_t)(ct0 + c) * NCB + cb) * T + t) * 64 + lane) * 4 + sl];
        }
        if (st > 0) __syncthreads();                      // every wave is done with the previous patch
        // (loads of NU units are in flight together.  Fetching the next stage's patch under the
        // multiplication instead, with the registers that takes, measured 5-15 % slower: the
        // workgroups that share a CU hide each other's loads)
        constexpr int NU = VEC ? 4 : 2;
        for (int k = 0; k < n_units; k += NU) {
            float v[NU][8];
#pragma unroll
            for (int u = 0; u < NU; ++u) load_unit(k + u, st, v[u]);
#pragma unroll
            for (int u = 0; u < NU; ++u) put_unit(k + u, st, v[u]);
        }
        if (KW == 1 && max_bits >= kMostBits) *whole_lds = 1;
        __syncthreads();
        if (KW == 1) whole = *whole_lds;                  // (looked at after the stage: its latency is covered)
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            const int s = kw + KW * j;
            if (KW > 1 && s >= STEPS) break;
            const int t = s / (KC / 16), sl = s % (KC / 16);
            // slice sl of the stage: the lane's 8 channels are group 2*h + (sl & 1) of half sl / 2
            const int off = ((t / R) * pl.PC + t % R) * (R == 1 ? 0 : PIXB) + (sl >> 1) * 64 + (sl & 1) * 16;
            v8bf xf[PF][3];
#pragma unroll
            for (int f = 0; f < PF; ++f)
#pragma unroll
                for (int p = 0; p < 3; ++p)
                    xf[f][p] = *reinterpret_cast<const v8bf *>(lds + frag_off[f] + off + p * KC * 2);
            v8bf wf[CT];
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                uint32_t b[2];
                dsq_unpack4(wreg[j][c], b[0], b[1]);
                seen |= wreg[j][c];
                v4i w;
                if constexpr (LUT) {
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const uint32_t lo = __builtin_amdgcn_perm(tab[c][1], tab[c][0], b[i]);
                        const uint32_t hi = __builtin_amdgcn_perm(tab[c][3], tab[c][2], b[i]);
                        w[2 * i] = (int)__builtin_amdgcn_perm(hi, lo, 0x05010400u);
                        w[2 * i + 1] = (int)__builtin_amdgcn_perm(hi, lo, 0x07030602u);
                    }
                } else
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float e0 = (float)((b[i >> 1] >> (16 * (i & 1))) & 0xFFu) + zq[c];
                    const float e1 = (float)((b[i >> 1] >> (16 * (i & 1) + 8)) & 0xFFu) + zq[c];
                    w[i] = (int)__builtin_amdgcn_perm(__float_as_uint(e1), __float_as_uint(e0), 0x07060302u);
                }
                wf[c] = __builtin_bit_cast(v8bf, w);
            }
#pragma unroll
            for (int p = 2; p >= 0; --p)                  // small terms first
#pragma unroll
                for (int c = 0; c < CT; ++c)
#pragma unroll
                    for (int f = 0; f < PF; ++f)
                        acc[f][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[c], xf[f][p], acc[f][c], 0, 0, 0);
        }
        // (the same in all waves; not with KW = 4, whose stages are as short as the look is long: 64 -> 70 us
        // for 4096->4096 x 64, and whose second pass is cheap.  Looking before the first stage's multiplication
        // as well made the 128x128 tile 10 % slower on NCHW tensors)
        if (KW == 1 && __builtin_amdgcn_readfirstlane(whole)) break;
    }
    // ---- epilogue -------------------------------------------------------------------
    // codes wider than the layer's bits are not on the grid of zq: such a tile is not split either
    if (max_bits >= kMostBits || (seen & ~((uint32_t)top * 0x11111111u))) *whole_lds = 1;
    float sx[PF];                                         // sum of x under the pixel's taps
#pragma unroll
    for (int f = 0; f < PF; ++f) sx[f] = 0.f;
    if (sums && T == 1) {
#pragma unroll
        for (int f = 0; f < PF; ++f)
#pragma unroll
            for (int g = 0; g < G; ++g) sx[f] += sx_lds[g * pl.npx + frag_pp[f]];
    } else if (sums) {
        // (a pixel's groups first: every tap of every pixel would add them up again)
        __syncthreads();
        for (int p = tid; p < pl.npx; p += 256) {
            float s = sx_lds[p];
#pragma unroll
            for (int g = 1; g < G; ++g) s += sx_lds[g * pl.npx + p];
            sx_lds[p] = s;
        }
        __syncthreads();
#pragma unroll
        for (int f = 0; f < PF; ++f)
#pragma unroll
            for (int t = 0; t < T; ++t) sx[f] += sx_lds[frag_pp[f] + (t / R) * pl.PC + t % R];
    }
    __syncthreads();                                      // the patch is free from here on
    const bool exact = __builtin_amdgcn_readfirstlane(*whole_lds) != 0;
    const size_t plane = (size_t)a.Ho * a.Wo;
    auto store4 = [&](int f, int o, const float (&v)[4]) {        // four consecutive channels of the lane's pixel
        if (frag_m[f] < 0) return;
        if (!a.out_nchw && (a.C_out & 3) == 0) {
            if (o < a.C_out) *reinterpret_cast<v4f *>(a.out + (size_t)frag_m[f] * a.C_out + o) = (v4f){v[0], v[1], v[2], v[3]};
            return;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (o + j < a.C_out) {
                if (a.out_nchw) a.out[((size_t)frag_n[f] * a.C_out + o + j) * plane + (size_t)frag_y[f] * a.Wo + frag_x[f]] = v[j];
                else a.out[(size_t)frag_m[f] * a.C_out + o + j] = v[j];
            }
    };
    if (exact) {                                          // (uniform over the workgroup)
        wq_exact_tiles<R, KW, PF, CT, VEC>(a, x, x_nchw, lane, kw, ct0, frag_m, frag_n, frag_y, frag_x, acc);
#pragma unroll
        for (int f = 0; f < PF; ++f) sx[f] = 0.f;
        if (tid < BC) { dw_lds[tid] = 1.0f; lr_lds[tid] = 0.f; }
        __syncthreads();
    }
    if constexpr (KW > 1) {
        // the partial tiles of the four waves meet in LDS; wave w finishes channels 8w + 4h ..
        v4f *part = reinterpret_cast<v4f *>(lds);         // [tile][wave][quarter][lane]
#pragma unroll
        for (int f = 0; f < PF; ++f)
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    part[(((f * CT + c) * KW + kw) * 4 + q) * 64 + lane] =
                        (v4f){acc[f][c][4 * q], acc[f][c][4 * q + 1], acc[f][c][4 * q + 2], acc[f][c][4 * q + 3]};
        __syncthreads();
#pragma unroll
        for (int f = 0; f < PF; ++f)
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                v4f s = part[((f * CT + c) * KW * 4 + kw) * 64 + lane];
#pragma unroll
                for (int w = 1; w < KW; ++w) s += part[(((f * CT + c) * KW + w) * 4 + kw) * 64 + lane];
                const int ol = c * 32 + 8 * kw + 4 * h;
                float v[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) v[j] = __builtin_fmaf(dw_lds[ol + j], s[j], lr_lds[ol + j] * sx[f]);
                store4(f, ct0 * 32 + ol, v);
            }
        return;
    }
    // NHWC: through this wave's slice of the idle patch area, so that a store
    // instruction writes 128 consecutive bytes of 8 pixels.  NCHW: 32 lanes already
    // hold 32 consecutive pixels of a channel.
    char *mine = lds + wave * (32 * ROWB);
    const bool staged = !a.out_nchw && (a.C_out & 3) == 0;
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        // (the channels' constants once for all fragments)
        float dw[16], lr[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int ol = (wc * CT + c) * 32 + 8 * (i / 4) + 4 * h + i % 4;
            dw[i] = dw_lds[ol];
            lr[i] = lr_lds[ol];
        }
#pragma unroll
        for (int f = 0; f < PF; ++f) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int ol = (wc * CT + c) * 32 + 8 * q + 4 * h;
                float v[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) v[j] = __builtin_fmaf(dw[4 * q + j], acc[f][c][4 * q + j], lr[4 * q + j] * sx[f]);
                if (staged) *reinterpret_cast<v4f *>(mine + col * ROWB + (8 * q + 4 * h) * 4) = (v4f){v[0], v[1], v[2], v[3]};
                else store4(f, blk_c * BC + ol, v);
            }
            if (staged) {
                // (LDS operations of one wave execute in order: no barrier needed)
                const int o = (ct0 + c) * 32 + (lane & 7) * 4;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int p = k * 8 + (lane >> 3);
                    const v4f t = *reinterpret_cast<const v4f *>(mine + p * ROWB + (lane & 7) * 16);
                    const int m = __shfl(frag_m[f], p);
                    if (m >= 0 && o < a.C_out) __builtin_nontemporal_store(t, reinterpret_cast<v4f *>(a.out + (size_t)m * a.C_out + o));
                }
            }
        }
    }
}

// ---- host side -------------------------------------------------------------------

template <int R, int WP, int WC, int KW, int PF, int CT, int OCC>
hipError_t launch(const DsqConvArgs &a, const float *x, int x_nchw, const WqPlan &pl, int lds, hipStream_t stream)
{
    const bool vec = !x_nchw && (a.C_in & 3) == 0;
    auto kern = a.bits <= 3 ? (vec ? conv_wq_kernel<R, WP, WC, KW, PF, CT, OCC, true, true> : conv_wq_kernel<R, WP, WC, KW, PF, CT, OCC, false, true>)
                            : (vec ? conv_wq_kernel<R, WP, WC, KW, PF, CT, OCC, true, false> : conv_wq_kernel<R, WP, WC, KW, PF, CT, OCC, false, false>);
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
    }
    kern<<<dim3(8 * pl.xcd_chunk), 256, lds, stream>>>(a, x, x_nchw, (1 << a.bits) - 1, pl);
    return hipGetLastError();
}

}  // namespace

// Tile by shape, from a sweep of every tile over 1x1 and 3x3 layers of 49 to 200704 pixels and
// 16 to 512 channels (us, tensors rotating over 700 MB, the tile named first against the one it
// was preferred to; the order is the same with the tensor in the last-level cache, 1 to 6 % less):
//   128x32   at most 32 output channels: nothing wider is filled (16->24 at 120x120 x 10: 20 against 25;
//            1x1 144->24 at 56x56 x 64 46 against 44)
//   32x32    K split over the four waves, fewer than 160 tiles of 64x64: the others leave most of the
//            chip idle (512->512 at 7x7 x 1: 32 against 55; level at 196 tiles, 18 against 19, and
//            behind from there, 128->128 at 28x28 x 16: 30 against 23)
//   128x128  layers that still give 192 of them, 3x3 stride 2 excepted: least staging, and least LDS
//            traffic per matrix instruction (128->128 at 28x28 x 64: 50 against 59, x 32 34 against 36;
//            1x1 256->512 stride 2 at 28x28 x 64: 23 against 28, 128->256 12 against 11)
//   64x128   3x3 stride 2: a patch of four times the pixels, staged for twice the channels
//            (64->128 at 56x56 x 64: 46 against 58)
//   64x64    the rest: four workgroups on a CU cover each other's staging, and the last round of
//            workgroups is short (128->128 at 28x28 x 8: 19 against 33 for 128x128)
hipError_t dsq_launch_conv_wq(const DsqConvArgs &a, const float *x, int x_nchw, hipStream_t stream)
{
    const long long M = (long long)a.N * a.Ho * a.Wo;
    auto blocks = [&](const WqTile &t) { return ((M + t.BP - 1) / t.BP) * ((a.C_out + t.BC - 1) / t.BC); };
    const bool wide = 4 * ((a.C_out + 127) / 128 * 128 - a.C_out) <= (a.C_out + 127) / 128 * 128;
    WqPlan pl;
    int lds = 0;
    if (blocks(kSquare) >= 160) {
        if (a.C_out <= 32 && plan_wq(a, kNarrow, pl, lds))
            return a.R == 3 ? launch<3, 4, 1, 1, 1, 1, 4>(a, x, x_nchw, pl, lds, stream)
                            : launch<1, 4, 1, 1, 1, 1, 4>(a, x, x_nchw, pl, lds, stream);
        if ((a.R == 1 || a.stride == 1) && wide && blocks(kLarge) >= 192 && plan_wq(a, kLarge, pl, lds))
            return a.R == 3 ? launch<3, 2, 2, 1, 2, 2, 2>(a, x, x_nchw, pl, lds, stream)
                            : launch<1, 2, 2, 1, 2, 2, 2>(a, x, x_nchw, pl, lds, stream);
        if (a.R == 3 && a.stride == 2 && wide && blocks(kRow) >= 320 && plan_wq(a, kRow, pl, lds))
            return launch<3, 2, 2, 1, 1, 2, 3>(a, x, x_nchw, pl, lds, stream);
        if (plan_wq(a, kSquare, pl, lds))
            return a.R == 3 ? launch<3, 2, 2, 1, 1, 1, 4>(a, x, x_nchw, pl, lds, stream)
                            : launch<1, 2, 2, 1, 1, 1, 4>(a, x, x_nchw, pl, lds, stream);
    }
    // (its patch fits for every geometry: 32 pixels of images of one output column and row, at
    // most 4 padded rows apart, are 32*4 rows of at most 4 columns)
    if (!plan_wq(a, kSplit, pl, lds)) return hipErrorInvalidValue;
    return a.R == 3 ? launch<3, 1, 1, 4, 1, 1, 4>(a, x, x_nchw, pl, lds, stream)
                    : launch<1, 1, 1, 4, 1, 1, 4>(a, x, x_nchw, pl, lds, stream);
}
