// Internal launch interface between the C ABI (api.hip) and the kernels.
// Arguments have already been validated by the caller.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#define DSQ_QUANT_MAX_PB 512   // most pixels one quantizer block may own

struct DsqConvArgs {
    int N, C_in, H, W, C_out, R, stride, pad, bits;
    int Ho, Wo;
    int cont;      // format of the packed activation codes: 2 or 4 = container width in bits,
                   // 3 = dense 3-bit units (weights are then in the 4-bit layout)
    int Cp;        // C_in rounded up to 64
    int Cop;       // C_out rounded up to 256
    const void *act;          // packed activation codes
    const int32_t *pix_sum;   // [N*H*W]
    float l_a, u_a;
    float delta_a;            // (u_a - l_a) / (2^bits - 1) in binary32, computed by the host
    int kernel;               // host only: DSQ_CONV_KERNEL value of the call (0 = automatic)
    int many_in_flight;       // host only: the caller keeps several calls in flight (DSQ_CONV_MANY_IN_FLIGHT)
    const void *wq;           // packed weights
    const float *delta_w;     // [Cop]
    const float *l_w;         // [Cop]
    const int32_t *sw_total;  // [Cop]
    const int32_t *sw_tap;    // [Cop][R*R]
    float *out;
    int32_t *acc;             // may be null
    int out_nchw;
    // chained mode (dsq_conv2d_requant): instead of out / acc the kernels write
    // the next layer's packed codes and add to its pixel code sums
    int rq;                   // 0 = plain fp32 output
    const float *rq_scale;    // [C_out] or null (= 1)
    const float *rq_shift;    // [C_out] or null (= 0)
    int rq_relu;
    float rq_l, rq_u;         // next layer's clip range
    int rq_bits;
    int rq_dense;             // next layer's codes in the dense 3-bit format (rq_bits == 3)
    float rq_delta;           // its step, the recipe's binary32 value
    // The LDS-patch kernel first decides a code in "code units":
    //   T = ((y*scale + shift) - l)/Delta,  code = clamp(T, rq_t_lo, rq_t_hi) rounded to nearest,
    // evaluated in binary32 from per-channel constants (conv_patch_kernel.h), and keeps
    // that code when T is farther from every half-integer than the error bound of the
    // evaluation; otherwise it falls back on the exact sequence above.  The host part
    // of that bound: rq_t_slack = 3*2^-24*(top + 1), what the recipe's three roundings
    // (subtraction, division, addition of 1/2) may move a value by, plus 2^-20 for
    // absolute rounding errors; rq_t_lo = 0, or code(0) under the ReLU; rq_t_hi = top;
    // rq_inv_dn = 1/Delta, rq_c0 = -l/Delta and rq_da_dn = Delta_a/Delta in binary64;
    // rq_sa_max bounds the sum of activation codes under one output, rq_w_max the
    // weight codes.  rq_fast = 0 (deep layers whose accumulators pass 2^24, extreme
    // ranges) sends every output through the exact sequence.
    int rq_fast;
    float rq_t_lo, rq_t_hi, rq_t_slack, rq_sa_max, rq_w_max;
    double rq_inv_dn, rq_c0, rq_da_dn;
    int rq_Cp;                // C_out rounded up to 64
    void *rq_codes;           // packed codes of the next layer's input
    int32_t *rq_pix;          // [N*Ho*Wo]; the kernels add to it (cleared before the launch) unless rq_store
    int rq_zeroed;            // the caller cleared rq_pix (DSQ_CONV_NEXT_SUMS_ZERO): launch no fill kernel
    int rq_share;             // set by a launcher: the waves of a workgroup add up their pixel sums in LDS first
    int rq_store;             // set by a launcher whose workgroups each hold all channels of their
                              // pixels: plain stores to rq_pix, nothing to clear
};

// The quantizer of one activation tensor.  With T(x) = (clip(x) - l)/Delta the recipe's code
// is T rounded to the nearest integer (halves up), but for values within
//   3*2^-24*(top + 1)
// of a half-integer, where its three roundings (subtraction, division, addition of 1/2) may
// decide; the kernels evaluate fma(clip(x), inv_delta, -l/Delta), which is within
//   2^-24*(max(|l|, |u|)/Delta + |l|/Delta + top + 3)
// of T (rounding of 1/Delta, of the constant and of the sum).  t_lo and t_hi are -l/Delta less
// and plus twice the sum of the two: where both round to the same integer, that is the
// recipe's code.  Ranges so far from 0 that the bound passes 1/4 get constants that never
// agree (t_lo = -1, t_hi = 2^8: codes 0 and 255), and run the recipe on every value.
struct DsqQuant {
    float l, u, delta;        // delta: the recipe's binary32 value
    float inv_delta, t_lo, t_hi;
    int top;
    int plain;                // the recipe has to divide (see quant4)
};

hipError_t dsq_launch_quantize_act(const float *x, int layout_nchw, int N, int C, int H, int W, int bits,
                                   const DsqQuant &q, void *codes, int32_t *pix_sum, hipStream_t stream);
// The same into the dense 3-bit format (bits == 3, C rounded up to 64 at most 8192).
hipError_t dsq_launch_quantize_act_dense3(const float *x, int layout_nchw, int N, int C, int H, int W, const DsqQuant &q,
                                          void *codes, int32_t *pix_sum, hipStream_t stream);

// `cont`: the container (2 or 4 bits) of the layer the weights are for; codes of
// `bits` <= cont bits are stored in it.
hipError_t dsq_launch_pack_weights(const float *w, const float *l_w, const float *u_w,
                                   const uint8_t *codes, int C_out, int C_in, int R, int bits, int cont,
                                   void *w_packed, void *w_aux, hipStream_t stream);

// Constants of the training-mode DSQ function for one tensor, computed on the
// host in binary64 and rounded once.
struct DsqSoftArgs {
    float l, u, delta, inv_delta;
    float last_interval;      // 2^b - 2
    float inv_levels;         // 1 / (2^b - 1)
    float k, s;
    float k_a, k_l, k_u;      // how k moves with alpha, l, u (0 when k is capped)
    float s_a, s_l, s_u;      // how s moves with alpha, l, u
};

hipError_t dsq_launch_soft_fwd(const float *x, float *y, size_t n, const DsqSoftArgs &p, hipStream_t stream);
hipError_t dsq_launch_soft_bwd(const float *x, const float *gy, float *gx, size_t n, const DsqSoftArgs &p,
                               double *sums, hipStream_t stream);

// Sets n int32 words to zero with a kernel (safe inside graph capture).
hipError_t dsq_launch_fill_zero(int32_t *p, size_t n, hipStream_t stream);

hipError_t dsq_launch_conv_simple(const DsqConvArgs &a, hipStream_t stream);
// force_tile: -1 = choose by problem size; 0 / 1 / 2 / 3 = the 128x64 / 128x128 /
// 256x128 / 256x64 (pixels x channels) workgroup tile.  Returns false, with nothing
// launched, if the LDS-patch kernel does not take this geometry with that tile;
// otherwise `status` is the launch's.
bool dsq_launch_conv_patch(const DsqConvArgs &a, int force_tile, hipStream_t stream, hipError_t &status);
// The launch configuration it would use, as text; returns 0 if it does not take the geometry.
int dsq_conv_patch_describe(const DsqConvArgs &a, int force_tile, char *text, size_t n);

// Split-K kernel for 1x1 layers with few output pixels (fully connected layers).
bool dsq_conv_fc_supported(const DsqConvArgs &a);   // the kernel takes this layer
bool dsq_conv_fc_preferred(const DsqConvArgs &a);   // ... and is the faster choice for it
hipError_t dsq_launch_conv_fc(const DsqConvArgs &a, hipStream_t stream);

// Split-K kernel for layers of few output tiles (one image or a few, of a small map).
bool dsq_conv_split_preferred(const DsqConvArgs &a);
hipError_t dsq_launch_conv_split(const DsqConvArgs &a, hipStream_t stream);

// Weight-only quantized layer: binary32 activations x (NHWC or NCHW), weights in the
// packed 4-bit layout; uses the geometry, wq, delta_w, l_w, out and out_nchw of `a`.
hipError_t dsq_launch_conv_wq(const DsqConvArgs &a, const float *x, int x_nchw, hipStream_t stream);
