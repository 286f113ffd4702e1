// Internal declarations of the sidelobe-network kernels (mlp_kernels.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#define MLP_IN 5
#define MLP_OUT 3
#define MLP_WCOL_ROWS 32   // rows of a block of the weighted column sums

namespace pisco {

#define MLP_MAX_L 16

// Fused inference + TOD epilogue over a pointing stream (infer_kernel).
struct MlpInferArgs {
    const double *th, *ph, *ps;  // pointing, n samples
    int64_t n;
    int32_t H, L;                // width, hidden layers
    const __bf16 *wb;            // bf16 parameter copy (first and last layer's weights)
    const __bf16 *wp;            // the hidden maps' weights, mlp_pack's fwd
    const float *w;              // fp32 parameters (biases used from it)
    int64_t off_w[MLP_MAX_L + 1], off_b[MLP_MAX_L + 1];
    float mean[3], stdv[3];
    double coef[3];
    float *tod;
};

hipError_t mlp_in_fwd(const float *x, const __bf16 *w0, const float *b0, int32_t n, int32_t H, float *z, __bf16 *a,
                      hipStream_t s);
// The H x H layers of a batch in one launch (chain_kernel), forward or backward.
struct MlpChain {
    const __bf16 *in;       // forward: A_0; backward: dZ_{L-1}; [rows][H]
    __bf16 *out;            // forward: A_{L-1}; backward: dZ_0
    const __bf16 *w;        // mlp_pack's W_1, W_2, ... (forward: fwd, backward: bwd)
    const float *bias;      // forward: b_1, b_2, ...
    int64_t b_stride;
    float *z;               // pre-activations [layer][rows][H], z_stride apart (forward: null = not stored)
    int64_t z_stride;
    __bf16 *t;              // transposed copies [layer][H][ldt]: forward A_0 .. A_{L-2} (null = not stored),
                            // backward dZ_{L-1} .. dZ_1
    int64_t t_stride, ldt;
    float *part_bias;       // backward: column sums of each layer's dZ, [layer][block of MLP_WCOL_ROWS rows][H]
    int64_t pb_stride;
    int32_t n, L, H;        // rows (buffers padded to 128), hidden layers, width
};
hipError_t mlp_chain(const MlpChain &c, bool bwd, int num_cu, hipStream_t s);
// partial[layer][slice] = A B over the slice's k_slice of the K rows of the batch, with
// A[m][k] at a[m*ld + k] and B(k, n) at b[n*ld + k]; the layers operand_stride and
// partial_stride apart.
hipError_t mlp_wgrad(const __bf16 *a, const __bf16 *b, int64_t ld, int64_t operand_stride, int32_t H, int32_t K,
                     int32_t k_slice, int32_t layers, float *partial, int64_t partial_stride, hipStream_t s);
// The H x H weights of `layers` maps (row-major, stride apart) in the fragment order of
// the kernels that multiply by them: fwd as they are, bwd transposed.
hipError_t mlp_pack(const __bf16 *src, int64_t stride, int32_t H, int32_t layers, __bf16 *fwd, __bf16 *bwd,
                    hipStream_t s);
// Fixed-order sums of several partial arrays in one launch.
#define MLP_MAX_SEGS 40
struct MlpReduceSeg {
    const float *part;
    float *out;
    int64_t count;
    int32_t slices;
    int32_t groups;   // slices summed in parallel groups (divides 256), combined in order
};
struct MlpReduceList {
    MlpReduceSeg seg[MLP_MAX_SEGS];
    int32_t n;
};
hipError_t mlp_reduce_many(const MlpReduceList &l, hipStream_t s);
hipError_t mlp_out(const __bf16 *a, const float *zL, const __bf16 *wout, const float *bout, int32_t n, int32_t H,
                   float *y, const float *tgt, float inv_count, float *dy, __bf16 *dz, float *part_loss,
                   int32_t waves, int32_t rows_per_wave, hipStream_t s);
// part[b * stride + u * su + k * sk] = sum over the rows r of block b (MLP_WCOL_ROWS
// rows each) of w(r, k) m[r][u], w(r, k) = wt[r K + k] or 1 (wt null, K = 1);
// ones[b K + k] = sum_r w(r, k) when given.  K in {1, 3, 5}.
hipError_t mlp_wcolsum(const __bf16 *m, const float *wt, int32_t K, int32_t n, int32_t H, float *part, int64_t stride,
                       int32_t su, int32_t sk, float *ones, hipStream_t s);
hipError_t mlp_adam(float *w, float *m, float *v, const float *g, __bf16 *wb, int64_t count, float lr_t, float b1,
                    float b2, float eps, float inv_bc2_sqrt, hipStream_t s);
hipError_t mlp_to_bf16(const float *w, __bf16 *wb, int64_t count, hipStream_t s);
hipError_t mlp_loss_sum(const float *part, int32_t count, float inv_count, float *loss, hipStream_t s);
hipError_t mlp_features(const double *th, const double *ph, const double *ps, int64_t n, float *x, hipStream_t s);
hipError_t mlp_infer_apply(const MlpInferArgs &a, hipStream_t s);
hipError_t mlp_apply(const float *y, int64_t n, const float *mean, const float *stdv, const double *coef, float *tod,
                     hipStream_t s);

}  // namespace pisco
