// dsq_quantize_act kernels: clip + round activations to b-bit codes (paper
// Algorithm 1 steps 1 and 3, i.e. the uniform quantizer of Sec. 3.1), pack
// them sub-byte and emit the per-pixel code sums the convolution epilogue
// needs for the l_w zero-point term.
//
// The kernels are bound by HBM traffic (4 B read and container/8 B written per
// element) as long as an element costs few vector instructions.  The recipe's IEEE
// division costs more than the memory time; looking the code up between two
// thresholds in LDS (a dozen instructions per element) still kept the vector units busy
// for 0.6 to 0.9 of the time.  Here (quant4) a code costs five instructions and a share
// of one comparison, and the recipe itself runs only where those cannot decide.
#include "dsq_device.h"
#include "dsq_kernels.h"

namespace {

template <int DPP_CTRL>
__device__ __forceinline__ int dpp_add(int v)
{
    return v + __builtin_amdgcn_update_dpp(0, v, DPP_CTRL, 0xF, 0xF, true);
}

template <int DPP_CTRL>
__device__ __forceinline__ uint32_t dpp_or(uint32_t v)
{
    return v | (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, DPP_CTRL, 0xF, 0xF, true);
}

// Codes of four values, one per byte.  T(x) = (clip(x) - l)/Delta is evaluated twice, a
// little below and a little above (q.t_lo and q.t_hi are -l/Delta -+ the error bound of
// this evaluation plus that of the recipe, see DsqQuant), and rounded to the nearest
// integer and packed by one instruction each (v_cvt_pk_u8_f32 rounds to nearest even).
// Where both agree, T is far enough from every midpoint for the recipe to give that code
// too.  Where a lane's do not (of ten thousand waves 5 / 13 / 26 / 50 at 1 / 2 / 3 / 4 bits, for the
// magnitudes of normally distributed values over a range that begins at 0; every time for values that
// sit on a midpoint, like 0 in a symmetric range), the wave runs the recipe: the quotient
// of the subtraction by Delta from a correctly rounded 1/Delta and two corrections by its exact
// remainder is the correctly rounded one (Markstein), so that nine instructions per value
// stand for the IEEE division's two dozen; only steps so small or large that a remainder
// might lose bits (q.plain) are divided.  A NaN gets code 0 as the last operand of
// v_med3_f32, which then returns min(min(l, u), x): l, or for a signalling NaN a quiet one,
// which converts to 0 (as the first operand it would give u).
// `active`: lanes whose values count (the others may hold anything).
__device__ __forceinline__ uint32_t quant4(float4 f, const DsqQuant &q, bool active)
{
    const float x[4] = {f.x, f.y, f.z, f.w};
    uint32_t lo = 0, hi = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float v = __builtin_amdgcn_fmed3f(q.l, q.u, x[j]);
        lo = __builtin_amdgcn_cvt_pk_u8_f32(__builtin_fmaf(v, q.inv_delta, q.t_lo), j, lo);
        hi = __builtin_amdgcn_cvt_pk_u8_f32(__builtin_fmaf(v, q.inv_delta, q.t_hi), j, hi);
    }
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(active && lo != hi) != 0, 0)) {
        if (q.plain) {
            asm volatile("");        // (a branch: left to itself the compiler computes both sides)
            return dsq_bytes4(dsq_code(x[0], q.l, q.u, q.delta, q.top), dsq_code(x[1], q.l, q.u, q.delta, q.top),
                              dsq_code(x[2], q.l, q.u, q.delta, q.top), dsq_code(x[3], q.l, q.u, q.delta, q.top));
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float s = __builtin_amdgcn_fmed3f(q.l, q.u, x[j]) - q.l;
            const float t0 = s * q.inv_delta;
            const float t1 = __builtin_fmaf(__builtin_fmaf(-t0, q.delta, s), q.inv_delta, t0);
            const float t = __builtin_fmaf(__builtin_fmaf(-t1, q.delta, s), q.inv_delta, t1);
            lo = __builtin_amdgcn_cvt_pk_u8_f32(floorf(t + 0.5f), j, lo);
        }
    }
    return lo;
}

// Codes of channels c..c+3 of a pixel whose channels lie `stride` floats apart; channels from C on
// are not read and have code 0.
__device__ __forceinline__ uint32_t quant4_of(const float *px, int stride, int c, int C, const DsqQuant &q)
{
    const int left = C - c;
    if (left <= 0) return 0u;
    px += (size_t)c * stride;
    float4 f = make_float4(px[0], 0.f, 0.f, 0.f);
    if (left > 1) f.y = px[stride];
    if (left > 2) f.z = px[2 * (size_t)stride];
    if (left > 3) f.w = px[3 * (size_t)stride];
    const uint32_t b = quant4(f, q, true);
    return left >= 4 ? b : b & ((1u << (8 * left)) - 1u);
}

// Sum of the four bytes of a word.
__device__ __forceinline__ int bytesum(uint32_t w) { return (int)__builtin_amdgcn_sad_u8(w, 0u, 0u); }

// NHWC input, C a multiple of 4 (and x 16-byte aligned, like every pointer of the
// library): rows of G lanes take a pixel each, lane r of a row the float4 units r, r + G,
// ... of it, so that a load instruction of a wave covers 64/G contiguous stretches.  From 16
// lanes on, those past the last channel make the code-0 padding; below, the words without a
// channel are written when the pixel is done.  The 2 (4-bit), 4 (2-bit) or 8
// (dense 3-bit) neighbouring lanes of a packed word combine their bytes with DPP moves.
// Code sums stay in the lanes until the pixel is done: no LDS, no atomics, no barrier.  A wave
// walks `steps` groups of 64/G pixels, the loads of U units in flight together.  4 bits, us, against
// a kernel that dealt float4 units to lanes block by block, looked codes up in LDS and added sums
// there (its vector units busy 0.9 of the time at 144 channels): 144 channels at 56x56 x 64 27.0 ->
// 23.5 (5.5 TB/s), 64 at 56x56 x 64 12.6 -> 10.8, 128 at 28x28 x 64 7.2 -> 5.2, 576 at 14x14 x 64 8.9 ->
// 6.9, 64 at 224x224 x 32 84 -> 78 (5.6 TB/s from HBM).
template <int CONT, int G, int U, bool NT>
__global__ __launch_bounds__(256) void quantize_act_rows_kernel(
    const float *__restrict__ x, uint32_t *__restrict__ codes, int32_t *__restrict__ pix_sum,
    int total_pixels, int C, int DP, int steps, DsqQuant q)
{
    constexpr bool D3 = CONT == 3;
    constexpr int LPW = D3 ? 8 : 8 / CONT;   // lanes per packed word (dense: per 12-byte unit)
    constexpr int WPG = D3 ? G / 8 * 3 : G / LPW;            // words of G units
    constexpr int PPS = 64 / G;              // pixels per step of a wave
    const int lane = threadIdx.x & 63, r = lane & (G - 1), row = lane / G;
    const int wave = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
    const int QP = C / 4;                                    // float4 units per pixel
    constexpr bool PADDED = G >= 16;
    // ... up to the end of the padding (a multiple of 16), or of the last word with a channel
    const int QPP = PADDED ? (D3 ? DP / 3 * 8 : DP * LPW) : (QP + LPW - 1) / LPW * LPW;
    const int J = (QPP + G - 1) / G;
    const int first = wave * steps * PPS;
    const int n = min(steps, (total_pixels - first + PPS - 1) / PPS);
    if (n <= 0) return;
    // (uniform bases, and 32-bit offsets of the lanes)
    const char *xb = (const char *)x + (size_t)first * QP * 16;
    uint32_t *cb = codes + (size_t)first * DP;
    const uint32_t x_row = (uint32_t)row * (uint32_t)QP * 16;
    const uint32_t c_off = (uint32_t)row * (uint32_t)DP + (D3 ? r / 8 * 3 + (lane & 7) : r / LPW);
    int sum = 0, j = 0, k = 0;               // unit j * G + r of pixel first + k * PPS + row
    while (k < n) {
        float4 f[U];
        int jl = j, kl = k;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            // Never under a branch: lanes without a unit read the first one of the row, lanes without
            // a pixel (of the last step) that of row 0, and past the last step the last one comes again
            const char *base = xb + ((size_t)kl * PPS * QP + (size_t)jl * G) * 16;
            const bool here = first + kl * PPS + row < total_pixels;
            const uint32_t off = (here ? x_row : 0u) + (jl * G + r < QP ? (uint32_t)r * 16 : 0u);
            if (NT) {
                // a tensor larger than the last-level cache is read once and never again
                typedef float v4f __attribute__((ext_vector_type(4)));
                const v4f t = __builtin_nontemporal_load(reinterpret_cast<const v4f *>(base + off));
                f[u] = make_float4(t.x, t.y, t.z, t.w);
            } else {
                f[u] = *reinterpret_cast<const float4 *>(base + off);
            }
            const bool wrap = jl + 1 == J;
            const int kn = wrap ? kl + 1 : kl, jn = wrap ? 0 : jl + 1;
            jl = kn < n ? jn : jl;
            kl = kn < n ? kn : kl;
        }
        __builtin_amdgcn_sched_barrier(0);       // (all loads first)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (u > 0 && k >= n) break;
            const int unit = j * G + r, pixel = first + k * PPS + row;
            const bool here = pixel < total_pixels, live = unit < QP && here;
            uint32_t b = quant4(f[u], q, live);
            b = live ? b : 0u;
            sum = (int)__builtin_amdgcn_sad_u8(b, 0u, (uint32_t)sum);
            uint32_t *out = cb + (size_t)k * PPS * DP + j * WPG;
            if (D3) {
                // lane g of a unit holds group g: its low bits go to word g / 4 at bit 2 (g % 4) of
                // every byte, its high bits to word 2 at bit g of every byte; the eight lanes OR
                // their shares together and lanes 0..2 store one word each
                const int g = lane & 7;
                const uint32_t low = (b & 0x03030303u) << (2 * (g & 3));
                uint32_t w0 = g < 4 ? low : 0u, w1 = g < 4 ? 0u : low, w2 = ((b >> 2) & 0x01010101u) << g;
                w0 = dpp_or<0x141>(dpp_or<0x4E>(dpp_or<0xB1>(w0)));
                w1 = dpp_or<0x141>(dpp_or<0x4E>(dpp_or<0xB1>(w1)));
                w2 = dpp_or<0x141>(dpp_or<0x4E>(dpp_or<0xB1>(w2)));
                if (g < 3 && unit < QPP && here) out[c_off] = g == 0 ? w0 : g == 1 ? w1 : w2;
            } else {
                uint32_t word;
                if (CONT == 4) {
                    // word = channels 8w..8w+7: byte j = c[j] | c[j+4] << 4; the odd lane holds c[4..7]
                    word = b | (uint32_t)__builtin_amdgcn_update_dpp(0, (int)b, 0xB1, 0xF, 0xF, true) << 4;
                } else {
                    // word = 16 channels: byte j = c[j] | c[j+4] << 2 | c[j+8] << 4 | c[j+12] << 6
                    word = dpp_or<0x4E>(dpp_or<0xB1>(b << (2 * (lane & 3))));
                }
                if ((lane & (LPW - 1)) == 0 && unit < QPP && here) out[c_off] = word;
            }
            if (j + 1 < J) {
                ++j;
            } else {
                int s = dpp_add<0xB1>(sum);                      // lanes ^1   (quad_perm 1,0,3,2)
                s = dpp_add<0x4E>(s);                            // lanes ^2   (quad_perm 2,3,0,1)
                if (G >= 8) s = dpp_add<0x141>(s);               // other quad (row_half_mirror)
                if (G >= 16) s = dpp_add<0x140>(s);              // other half row (row_mirror)
                if (G == 64)
                    s = __builtin_amdgcn_readlane(s, 0) + __builtin_amdgcn_readlane(s, 16) + __builtin_amdgcn_readlane(s, 32) +
                        __builtin_amdgcn_readlane(s, 48);
                if (r == 0 && here) pix_sum[pixel] = s;
                if (!PADDED && here)
                    for (int d = (D3 ? QPP / 8 * 3 : QPP / LPW) + r; d < DP; d += G)
                        (cb + ((size_t)k * PPS + row) * DP)[d] = 0;
                sum = 0;
                j = 0;
                ++k;
            }
        }
    }
}

// NHWC input with any number of channels.  One thread produces one packed word (8 channels
// at 4-bit, 16 at 2-bit).  A block owns PB whole pixels, so pixel sums never straddle blocks.
// Because a pixel is a multiple of 8 (4-bit) or 4 (2-bit) words long and the
// block starts on a pixel, every aligned group of 8 (4) lanes works on one
// pixel: their code sums are combined with DPP adds before one lane either
// stores the pixel sum (one group per pixel) or adds it into LDS.
template <int CONT>
__global__ __launch_bounds__(256) void quantize_act_nhwc_kernel(
    const float *__restrict__ x, uint32_t *__restrict__ codes, int32_t *__restrict__ pix_sum,
    int total_pixels, int C, int DP, int dp_shift, int PB, DsqQuant q)
{
    constexpr int CPD = 32 / CONT;           // channels per packed word
    constexpr int GROUP = CPD == 8 ? 8 : 4;  // lanes that surely share a pixel
    __shared__ int spix[DSQ_QUANT_MAX_PB];
    const int tid = threadIdx.x;
    const int pixel0 = blockIdx.x * PB;
    const int npix = min(PB, total_pixels - pixel0);
    const bool multi_group = DP != GROUP;
    if (multi_group) {
        for (int i = tid; i < npix; i += 256) spix[i] = 0;
        __syncthreads();
    }
    const int ndw = npix * DP;
    const int ndw_up = (ndw + 255) & ~255;   // all lanes take part in the DPP adds

    for (int i = tid; i < ndw_up; i += 256) {
        const bool active = i < ndw;
        const int p = dp_shift >= 0 ? (i >> dp_shift) : (i / DP);
        const int d = i - p * DP;
        const int c0 = d * CPD;
        uint32_t word = 0;
        int s = 0;
        if (active) {
            const float *px = x + (size_t)(pixel0 + p) * C;
#pragma unroll
            for (int g = 0; g < CPD / 4; ++g) {
                const uint32_t b = quant4_of(px, 1, c0 + 4 * g, C, q);
                word |= b << (CONT * g);
                s += bytesum(b);
            }
            codes[(size_t)(pixel0 + p) * DP + d] = word;
        }
        s = dpp_add<0xB1>(s);                    // lanes ^1   (quad_perm 1,0,3,2)
        s = dpp_add<0x4E>(s);                    // lanes ^2   (quad_perm 2,3,0,1)
        if (GROUP == 8) s = dpp_add<0x141>(s);   // other quad (row_half_mirror)
        if (active && (tid & (GROUP - 1)) == 0) {
            if (multi_group) atomicAdd(&spix[p], s);
            else pix_sum[pixel0 + p] = s;
        }
    }
    if (multi_group) {
        __syncthreads();
        for (int i = tid; i < npix; i += 256) pix_sum[pixel0 + i] = spix[i];
    }
}

// NHWC input of few, deep pixels (the input of a fully connected layer): a block of 256 or 1024
// threads owns one pixel, and a thread has the loads of U packed words in flight.  Words past
// the pixel's end are neither loaded nor quantized (with them 8192 channels, a quarter of the
// large block's words, took 6.4 us at 64 pixels).  Bound by the latency of the 4*C bytes that one
// compute unit reads.  C is a multiple of 4.
template <int CONT, int THREADS>
__global__ __launch_bounds__(THREADS) void quantize_act_deep_kernel(const float *__restrict__ x, uint32_t *__restrict__ codes,
                                                                 int32_t *__restrict__ pix_sum, int C, int DP, DsqQuant q)
{
    constexpr int CPD = 32 / CONT, FPW = CPD / 4;    // channels and float4 groups per packed word
    constexpr int U = 8 / FPW;
    __shared__ int part[THREADS / 64];
    const int tid = threadIdx.x;
    const float *px = x + (size_t)blockIdx.x * C;
    uint32_t *row = codes + (size_t)blockIdx.x * DP;
    int sum = 0;
    for (int base = tid; base < DP; base += THREADS * U) {
        float4 f[U][FPW];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            if (base + k * THREADS >= DP) continue;     // (whole waves, but for the one that holds the pixel's end)
#pragma unroll
            for (int g = 0; g < FPW; ++g) {
                const int c = (base + k * THREADS) * CPD + 4 * g;
                f[k][g] = *reinterpret_cast<const float4 *>(px + (c < C ? c : 0));      // (blanked below)
            }
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int d = base + k * THREADS;
            if (d >= DP) continue;
            uint32_t word = 0;
#pragma unroll
            for (int g = 0; g < FPW; ++g) {
                const bool in = d * CPD + 4 * g < C;
                const uint32_t b = quant4(f[k][g], q, in), m = in ? b : 0u;
                word |= m << (CONT * g);
                sum += bytesum(m);
            }
            row[d] = word;
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_down(sum, off);
    if ((tid & 63) == 0) part[tid >> 6] = sum;
    __syncthreads();
    if (tid == 0) {
        int s = 0;
#pragma unroll
        for (int w = 0; w < THREADS / 64; ++w) s += part[w];
        pix_sum[blockIdx.x] = s;
    }
}

// NCHW input.  Lanes run along 64 pixels of one image plane (contiguous in memory for a
// fixed channel); the NW waves of a block take the packed words of those pixels in turn.
// The words of up to 64 per pixel meet in LDS, from where the block writes them out as the
// contiguous run that 64 pixels of the packed tensor are (lanes that store one word each
// touch 64 separate rows per instruction).  4 bits, us, with the codes looked up between
// thresholds in LDS -> now (tensor in the last-level cache): 128 channels at 28x28 x 64 9.5 -> 7.9,
// 512 at 7x7 x 64 8.3 -> 6.5, 64 at 56x56 x 64 13.2 -> 11.2.
template <int CONT, int NW>
__global__ __launch_bounds__(64 * NW) void quantize_act_nchw_kernel(
    const float *__restrict__ x, uint32_t *__restrict__ codes, int32_t *__restrict__ pix_sum,
    int C, int HW, int DP, DsqQuant q)
{
    constexpr int CPD = 32 / CONT;
    constexpr int MOST = 64;                         // words per pixel and pass
    __shared__ uint32_t words[64 * (MOST + 1)];      // (odd row length: no bank conflicts)
    __shared__ int ssum[NW][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int hw0 = blockIdx.x * 64;
    const int npix = min(64, HW - hw0);
    const int n = blockIdx.y;
    const float *xn = x + (size_t)n * C * HW + hw0 + min(lane, npix - 1);
    const size_t pixel0 = (size_t)n * HW + hw0;
    int s = 0;
    for (int d0 = 0; d0 < DP; d0 += MOST) {
        const int nd = min(MOST, DP - d0);           // a multiple of 4, like DP
        // words without a channel (7 of 8 where there are three channels) are neither loaded nor quantized
        const int live = min(nd, (C - d0 * CPD + CPD - 1) / CPD);
        for (int d = wave; d < live; d += NW) {
            const int c0 = (d0 + d) * CPD;
            float v[CPD];
#pragma unroll
            for (int j = 0; j < CPD; ++j) v[j] = xn[(size_t)(c0 + j < C ? c0 + j : 0) * HW];
            uint32_t word = 0;
            // channel j of the word sits in byte j%4 at bit offset CONT*(j/4)
#pragma unroll
            for (int g = 0; g < CPD / 4; ++g) {
                const int left = C - (c0 + 4 * g);           // (uniform)
                if (left <= 0) break;
                uint32_t b = quant4(make_float4(v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]), q, true);
                if (left < 4) b &= (1u << (8 * left)) - 1u;
                word |= b << (CONT * g);
                s += bytesum(b);
            }
            words[lane * (MOST + 1) + d] = word;
        }
        for (int d = max(live, 0) + wave; d < nd; d += NW) words[lane * (MOST + 1) + d] = 0;
        __syncthreads();
        const int quads = nd / 4;
        for (int i = tid; i < npix * quads; i += 64 * NW) {
            const int p = i / quads, d = 4 * (i - p * quads);
            const uint32_t *w = words + p * (MOST + 1) + d;
            *reinterpret_cast<uint4 *>(codes + (pixel0 + p) * DP + d0 + d) = make_uint4(w[0], w[1], w[2], w[3]);
        }
        if (d0 + MOST < DP) __syncthreads();         // before the next pass overwrites the words
    }
    ssum[wave][lane] = s;
    __syncthreads();
    if (tid < npix) {
        int t = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) t += ssum[w][tid];
        pix_sum[pixel0 + tid] = t;
    }
}

// ---- dense 3-bit output ---------------------------------------------------------
// 32 channels of a pixel become one 12-byte unit (format: dsq_device.h).
//
// NHWC, any number of channels: one thread per unit, the units of a pixel in neighbouring
// lanes; a block owns whole pixels (PB of them, UPX units each) and adds up their code sums in LDS.
__global__ __launch_bounds__(256) void quantize_act_dense3_nhwc_kernel(const float *__restrict__ x, uint32_t *__restrict__ codes,
                                                                       int *__restrict__ pix_sum, int pixels, int C, int UPX,
                                                                       int PB, DsqQuant q)
{
    __shared__ int psum[256];
    const int tid = threadIdx.x;
    psum[tid] = 0;
    __syncthreads();
    const int pl = tid / UPX, k = tid - pl * UPX;
    const long long p = (long long)blockIdx.x * PB + pl;
    if (pl < PB && p < pixels) {
        const float *row = x + (size_t)p * C;
        uint32_t d[8];
        int sum = 0;
#pragma unroll
        for (int g = 0; g < 8; ++g) {
            d[g] = quant4_of(row, 1, 32 * k + 4 * g, C, q);
            sum += bytesum(d[g]);
        }
        uint32_t l0, l1, hi;
        dsq_pack32_d3(d, l0, l1, hi);
        uint32_t *w = codes + ((size_t)p * UPX + k) * 3;
        w[0] = l0; w[1] = l1; w[2] = hi;
        atomicAdd(&psum[pl], sum);
    }
    __syncthreads();
    if (tid < PB && (long long)blockIdx.x * PB + tid < pixels) pix_sum[(long long)blockIdx.x * PB + tid] = psum[tid];
}

// NCHW: one thread per pixel (neighbouring lanes = neighbouring pixels of a row, so the
// reads of a channel are contiguous); the thread walks the pixel's units.
__global__ __launch_bounds__(256) void quantize_act_dense3_nchw_kernel(const float *__restrict__ x, uint32_t *__restrict__ codes,
                                                                       int *__restrict__ pix_sum, int C, int HW, int UPX,
                                                                       DsqQuant q)
{
    const int hw = blockIdx.x * 256 + threadIdx.x;
    const int n = blockIdx.y;
    if (hw >= HW) return;
    const float *img = x + (size_t)n * C * HW + hw;
    const size_t p = (size_t)n * HW + hw;
    int sum = 0;
    for (int k = 0; k < UPX; ++k) {
        uint32_t d[8];
#pragma unroll
        for (int g = 0; g < 8; ++g) {
            d[g] = quant4_of(img, HW, 32 * k + 4 * g, C, q);
            sum += bytesum(d[g]);
        }
        uint32_t l0, l1, hi;
        dsq_pack32_d3(d, l0, l1, hi);
        uint32_t *w = codes + (p * UPX + k) * 3;
        w[0] = l0; w[1] = l1; w[2] = hi;
    }
    pix_sum[p] = sum;
}

// Rows of 4 to 64 lanes, units in flight, and steps per wave.  All figures in us, 4 bits unless stated, tensor in the
// last-level cache where it fits.
template <int CONT>
void launch_rows(const float *x, uint32_t *codes, int32_t *pix_sum, int total_pixels, int C, int DP, const DsqQuant &q,
                 hipStream_t stream)
{
    const int QP = C / 4, units = dsq_round_up(C, 64) / 4;
    // 64 lanes where a pixel has as many units and there are few of them: 4 / 8 / 16 / 64 lanes take 11.4 / 6.9
    // / 4.6 / 3.1 for 512 channels at 7x7 x 64, but at 64 channels, 56x56 x 64, 12.6 / 11.0 / 11.1 / 24.9 (with
    // more loads than this the 16-lane rows are level or ahead).  However many there are where a 16-lane row would
    // walk a pixel in twelve steps: 16 / 64 lanes 768 channels at 14x14 x 64 9.8 / 7.9, 1024 12.4 / 10.6, 1536 17.1 / 14.5.
    // And 48 units where the lanes fit the chip at once: 192 channels at 28x28 x 1 2.89 / 2.43, x 4 2.94 / 2.64.
    // Below 16 units a row of 16 is mostly
    // idle: 16 channels at 56x56 x 64 4.9 / 6.3 / 8.4, 40 channels 8.8 / 9.1 / 9.1; 80 channels at 73x73 x
    // 16 7.4 / 6.8 / 7.8.  But a small tensor takes as long as a lane has steps: 4 / 8 lanes 32 channels at 28x28 x 1
    // 2.57 / 2.39, x 8 2.62 / 2.43, 56x56 x 16 3.15 / 3.26; 48 at 28x28 x 1 4 / 8 / 16 2.79 / 2.56 / 2.4.  (From 2^24
    // channels on the offsets of a row of pixels would not fit 32 bits.)
    const long long loads = (long long)total_pixels * units / 64, all_units = (long long)total_pixels * QP;
    const bool small = all_units < 128 * 1024;
    const int G = C >= (1 << 24) || (units >= 64 && loads < 32768) || (units >= 48 && loads < 4096) || units >= 192 ? 64
                : QP <= (small ? 4 : 12) && CONT != 3 ? 4 : QP == 16 || QP >= 24 || (small && QP > 8) ? 16 : 8;
    // Tensors of 192 MB and more (three quarters of the last-level cache) are read with
    // non-temporal loads, in long waves with four in flight: 224x224 x 64 channels x 32 78 us, 88 with one in
    // flight and two steps; 112x112 x 128 x 32 41, with one in flight 44.  Smaller tensors: two loads a wave
    // (112x112 x 64 x 32 18.2, with one 19.3, with eight 19.1), one where that leaves the chip short of waves.
    const bool nt = all_units >= 12LL * 1024 * 1024;
    const int pps = 64 / G, J = G >= 16 ? (units + G - 1) / G : (QP + G - 1) / G;
    // Large tensors whose pixels are three units a lane: all three in flight together, two pixels a wave and row.  us, one
    // (four, non-temporal) in flight / three: 144 channels at 56x56 x 64 24.1 / 22.2, 2 bits 22.7 / 21.6 (58 MB of them 13.5 /
    // 13.0, but 43 MB 10.5 / 11.0), x 128 57.2 / 51.9, 2 bits 54.2 / 49.8, 192 channels x 128 65.5 / 60.5; rows of 8, 72
    // channels x 64 16.2 / 13.8, 2 bits 14.5 / 13.3, 80 16.1 / 14.2, 2 bits 14.9 / 13.7.  Not where the third
    // unit is one for nearly all lanes: 176 channels x 64 2 bits 24.5 / 24.8, 192 25.2 / 25.6.
    // Rows of 4 lanes with more than one unit a lane: four, some of them twice.  32 channels at 56x56 x 128 13.1 /
    // 12.2, 2 bits 12.5 / 11.1, 48 18.1 / 15.4, 2 bits 16.8 / 14.9, but at half the pixels 6.1 / 7.2 (32).
    const bool large = all_units >= 3LL * 1024 * 1024;
    const bool three = large && J == 3 && (G == 8 || (G == 16 && (nt || QP <= 40))), four = large && G == 4 && J > 1;
    int steps = three ? 2 : four ? 1 : (nt ? 8 : 2) / J;
    while (!three && steps > 1 && (long long)total_pixels / (pps * steps) < 8192) steps >>= 1;
    if (steps < 1) steps = 1;
    const long long waves = ((long long)total_pixels + pps * steps - 1) / (pps * steps);
    const dim3 grid((unsigned)((waves + 3) / 4));
#define DSQ_ROWS(G, U, NT) quantize_act_rows_kernel<CONT, G, U, NT><<<grid, 256, 0, stream>>>(x, codes, pix_sum, total_pixels, C, DP, steps, q)
    if (G == 64 && nt) DSQ_ROWS(64, 4, true);
    else if (G == 64) DSQ_ROWS(64, 1, false);
    else if (G == 8 && three) DSQ_ROWS(8, 3, false);
    else if (G == 8) DSQ_ROWS(8, 1, false);
    else if (G == 16 && three && nt) DSQ_ROWS(16, 3, true);
    else if (G == 16 && three) DSQ_ROWS(16, 3, false);
    else if (G == 16 && nt) DSQ_ROWS(16, 4, true);
    else if (G == 16) DSQ_ROWS(16, 1, false);
    else if constexpr (CONT != 3) {
        if (four) DSQ_ROWS(4, 4, false);
        else DSQ_ROWS(4, 1, false);
    }
#undef DSQ_ROWS
}

}  // namespace

hipError_t dsq_launch_quantize_act(const float *x, int layout_nchw, int N, int C, int H, int W, int bits,
                                   const DsqQuant &q, void *codes, int32_t *pix_sum, hipStream_t stream)
{
    const int cont = dsq_container(bits);
    const int DP = dsq_round_up(C, 64) * cont / 32;
    const int total_pixels = N * H * W;
    uint32_t *cw = (uint32_t *)codes;
    // (one pixel per image: the two layouts are the same memory)
    if (layout_nchw && H * W > 1) {
        dim3 grid((H * W + 63) / 64, N);
        // 16 waves per block on tensors that do not fill the chip with four each, unless that leaves
        // waves without a word.  us, four / 16 waves, 4 bits: 128 channels (16 words) at 14x14 x 64 6.6 /
        // 4.6, 28x28 x 64 (832 blocks) 10.1 / 9.8, 56x56 x 64 (3136 blocks) 21.8 / 25.6, 112x112 x 32 (6272)
        // 37 / 45; 512 channels 21.9 / 10.7 at 14x14 x 64, 95 / 89 at 56x56 x 64.  So from about 1000 blocks
        // on pixels of 16 to 24 words are up to 20 % better off with four, deeper ones with 16.
        const bool many = DP >= 16 && (long long)grid.x * grid.y < 4096;
#define DSQ_NCHW_LAUNCH(CONT, NW) quantize_act_nchw_kernel<CONT, NW><<<grid, 64 * NW, 0, stream>>>(x, cw, pix_sum, C, H * W, DP, q)
        if (cont == 4) { if (many) DSQ_NCHW_LAUNCH(4, 16); else DSQ_NCHW_LAUNCH(4, 4); }
        else           { if (many) DSQ_NCHW_LAUNCH(2, 16); else DSQ_NCHW_LAUNCH(2, 4); }
#undef DSQ_NCHW_LAUNCH
        return hipGetLastError();
    }
    if (C % 4 == 0) {
        // A block per pixel where pixels are deep (us, 4 bits, a wave of the rows kernel per pixel / blocks
        // of 256 / of 1024 threads): 4096 channels x 1 5.7 / 2.5 / 2.4, x 64 6.7 / 2.8 / 2.8, x 600 6.6 / 3.6 / 4.0, x 3136
        // 12.2 / 10.6 / 11.6, x 12544 35 / 34.6 / 36; 2048 x 6272 10.4 / 10.5 / 17.7 (16 lanes of the rows kernel 19.2), x 25088
        // 34 / 33.9 / 61.  1024 threads from 8192 (2 bits: 16384) channels on, of which 512 blocks run at a time: 8192 x 784
        // 4.8 / 5.4 (256 / 1024 threads), x 4096 24.2 / 23.9 / 22.1, x 12544 85 / 86 / 81.  Few pixels from 768 channels
        // on: 768 x 512 2.85 / 2.68, x 3136 3.53 / 4.10, 1024 x 49 3.16 / 2.63, x 784 3.25 / 2.86, x 1568 3.37 / 3.20,
        // x 3136 3.96 / 4.10 / 8.4.
#define DSQ_DEEP(T) do { if (cont == 4) quantize_act_deep_kernel<4, T><<<total_pixels, T, 0, stream>>>(x, cw, pix_sum, C, DP, q); \
            else quantize_act_deep_kernel<2, T><<<total_pixels, T, 0, stream>>>(x, cw, pix_sum, C, DP, q); } while (0)
        if (DP >= 1024 && (total_pixels <= 512 || total_pixels >= 2048)) {
            DSQ_DEEP(1024);
        } else if (C >= 2048 || (C >= 1024 && total_pixels <= 2048) || (C >= 768 && total_pixels <= 512)) {
            DSQ_DEEP(256);
        } else if (cont == 4) {
            launch_rows<4>(x, cw, pix_sum, total_pixels, C, DP, q, stream);
        } else {
            launch_rows<2>(x, cw, pix_sum, total_pixels, C, DP, q, stream);
        }
#undef DSQ_DEEP
        return hipGetLastError();
    }
    // Words per thread: few for small tensors (enough blocks to cover the
    // chip), more for large ones (more loads in flight per thread).
    const long long total_dw = (long long)total_pixels * DP;
    int iters = 8;
    while (iters > 1 && total_dw / (256LL * iters) < 2048) iters >>= 1;
    int PB = (256 * iters) / DP;
    if (PB < 1) PB = 1;
    if (PB > DSQ_QUANT_MAX_PB) PB = DSQ_QUANT_MAX_PB;
    int dp_shift = -1;
    if ((DP & (DP - 1)) == 0) { dp_shift = 0; while ((1 << dp_shift) < DP) ++dp_shift; }
    dim3 grid((total_pixels + PB - 1) / PB);
    if (cont == 4) quantize_act_nhwc_kernel<4><<<grid, 256, 0, stream>>>(x, cw, pix_sum, total_pixels, C, DP, dp_shift, PB, q);
    else quantize_act_nhwc_kernel<2><<<grid, 256, 0, stream>>>(x, cw, pix_sum, total_pixels, C, DP, dp_shift, PB, q);
    return hipGetLastError();
}

hipError_t dsq_launch_quantize_act_dense3(const float *x, int layout_nchw, int N, int C, int H, int W, const DsqQuant &q,
                                          void *codes, int32_t *pix_sum, hipStream_t stream)
{
    const int UPX = dsq_round_up(C, 64) / 32;        // units per pixel (<= 256: checked by the caller)
    const int pixels = N * H * W;
    if (layout_nchw) {
        dim3 grid((H * W + 255) / 256, N);
        quantize_act_dense3_nchw_kernel<<<grid, 256, 0, stream>>>(x, (uint32_t *)codes, pix_sum, C, H * W, UPX, q);
    } else if (C % 4 == 0) {
        launch_rows<3>(x, (uint32_t *)codes, pix_sum, pixels, C, UPX * 3, q, stream);
    } else {
        const int PB = 256 / UPX;
        quantize_act_dense3_nhwc_kernel<<<(pixels + PB - 1) / PB, 256, 0, stream>>>(x, (uint32_t *)codes, pix_sum,
                                                                                    pixels, C, UPX, PB, q);
    }
    return hipGetLastError();
}
