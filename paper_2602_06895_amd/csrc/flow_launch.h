// Host-side launchers of the coupling-flow kernels (defined in flow_kernels.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace msx {

constexpr int kFlowMaxBins = 32;   // spline bins per coordinate
constexpr int kFlowMaxHalf = 32;   // transformed coordinates per layer (dims / 2)

// Element type of the MLP operands on the matrix cores.
enum FlowType : int { FT_BF16 = 0, FT_F32 = 1 };

// Epilogue of a GEMM tile.
enum GemmEpi : int {
    EPI_PARTIAL = 0,    // out_f32[z][m][n] = acc (split-K partial sums)
    EPI_BIAS_RELU = 1,  // out_t[m][n] = T(max(acc + bias[n], 0))
    EPI_BIAS_F32 = 2,   // out_f32[m][n] = acc + bias[n]
    EPI_RELU_MASK = 3,  // out_t[m][n] = T(mask[m][n] > 0 ? acc : 0)
    EPI_F32 = 4         // out_f32[m][n] = acc
};

// C[M][N] (+ epilogue) = sum_k A(m, k) B(k, n) with A(m, k) = A[m a_m + k a_k]
// and B(k, n) = B[k b_k + n b_n] (one of the two strides of each operand is
// 1).  `splits` > 1 divides K into that many chunks (EPI_PARTIAL only).
struct GemmArgs {
    int type;  // FlowType of A, B, out_t and mask
    int M, N, K;
    const void* A;
    int64_t a_m, a_k;
    const void* B;
    int64_t b_k, b_n;
    int splits;
    int epi;
    void* out;
    int64_t ldc;
    const float* bias;
    const void* mask;
    int64_t ldm;
};
hipError_t launch_gemm(const GemmArgs& g, hipStream_t s);

// Coupling layers of hidden width 128 and up to 16 bins have kernels of their
// own: conditioner on the matrix cores and spline together.
constexpr int kFusedHidden = 128;
constexpr int kFusedMaxBins = 16;

// Parameters of a flow with such layers: the operand copy (BF16, or FP32 if
// f32; layer blocks of per_t elements, 16-byte aligned), the FP32 parameters
// (blocks of per), and the offsets of W1 b1 W2 b2 W3 b3 W4 b4 in both.
struct FlowNet {
    const void* wt;
    const float* p;
    int32_t per_t, per;
    int32_t off[8];
    int32_t nh, K, f32;
};
// A pass over `count` layers first, first + dir, ...: n events [d][n] from
// zin; the i-th layer of the pass leaves its result in zout + i zstep (zstep
// 0: one buffer, which may be zin).  logdet [n] receives the sum of the
// layers' log-determinants.
struct FlowRun {
    const float* zin;
    float* zout;
    int64_t zstep;
    float* logdet;
    int64_t n;
    int first, dir, count;
};
hipError_t launch_flow_layers(bool inverse, const FlowNet& fn, const FlowRun& run, int cu_count, hipStream_t s);

// Reverse mode of one inverse layer of such a flow.  The matrices between its
// kernels, of the operands' type, are in blocks of 32 events, [blocks][rows][32],
// which is how the weight gradients read them: an operand of 16 rows and 32
// events has no gaps.  Whole tiles of up to 64 events are written; columns
// beyond n of d and dh are zero.
struct FlowRev {
    const float* zin;  // the layer's input [d][n], before inversion
    float* adj;        // [d][n] adjoint, of the layer's output on entry, of its input on exit
    const float* G;    // [n] dLoss/dlogq
    void* x0;          // [blocks][32][32] conditioning inputs (rows beyond nh undefined)
    void* h;           // [blocks][3 * 128][32] hidden activations
    uint16_t* on;      // [tiles of at least 32 events][3][512] which of them are positive
    void* d;           // [blocks][flow_grad_rows][32] gradients of the spline parameters
    void* dh;          // [blocks][3 * 128][32] gradients of the hidden layers before their ReLU
    int64_t n;
    int layer;
    int first;         // adj counts as zero on entry
};
// Rows of FlowRev::d (the last ones undefined).
int flow_grad_rows(int nh, int K);
// Hidden activations and spline recomputed, spline reversed: fills x0, h, on,
// d and the transformed coordinates of adj.
hipError_t launch_flow_spline_reverse(const FlowNet& fn, const FlowRev& r, int cu_count, hipStream_t s);
// Transposed weights of all layers, for the next call: wt_t holds
// flow_transposed_elems(nh) elements per layer.
int64_t flow_transposed_elems(int nh);
hipError_t launch_flow_transpose(const FlowNet& fn, int layers, void* wt_t, hipStream_t s);
// Through the conditioner: fills dh and the conditioning coordinates of adj.
hipError_t launch_flow_mlp_reverse(const FlowNet& fn, const FlowRev& r, const void* wt_t, int cu_count,
                                   hipStream_t s);
// Weight and bias gradients of the layer from d, dh, h, x0: partial sums over
// `splits` runs of events, part [splits][per], laid out as the parameters.
int flow_wgrad_splits(const FlowNet& fn, int64_t n);
hipError_t launch_flow_wgrad(const FlowNet& fn, const FlowRev& r, int splits, float* part, int cu_count,
                             hipStream_t s);

// out[m][n] = sum_z part[z][m][n] in z order (out has leading dimension ldo).
hipError_t launch_reduce_partials(const float* part, int splits, int M, int N, float* out, int64_t ldo,
                                  hipStream_t s);

// Column sums of an [R][N] matrix of type `type` (bias gradients), written to
// out[N]; `part` holds at least nchunk * N floats.
hipError_t launch_colsum(int type, const void* X, int64_t R, int N, int64_t ldx, float* part, int nchunk, float* out,
                         hipStream_t s);

// X0[b][i] = T(z[cond[i]][b]) for the conditioning coordinates of a layer.
hipError_t launch_gather(int type, const float* z, int64_t n, int n_cond, const int32_t* cond_host, void* x0,
                         hipStream_t s);

// Spline of every transformed coordinate of one layer, one thread per
// (event, coordinate).
//   forward: z[t_j] <- S(z[t_j]), logdet += sum_j log S'
//   inverse: z[t_j] <- S^-1(z[t_j]), logdet += sum_j log (S^-1)'
// ld_part: scratch of n_half x n floats (the per-coordinate terms).
hipError_t launch_spline(bool inverse, float* z, int64_t n, const float* theta, int64_t ldt, int n_half,
                         const int32_t* trans_host, int K, float* logdet, float* ld_part, hipStream_t s);

// Reverse mode through one inverse spline layer.  y: layer input (its
// transformed coordinates, before inversion), adj: adjoint of the layer output
// on entry, of the layer input on exit (transformed coordinates; conditioning
// coordinates are left for launch_scatter_add), G[b] = dLoss/dlogq_b.  Writes
// dtheta (type `type`, leading dimension ldt).
hipError_t launch_spline_backward(int type, const float* y, float* adj, int64_t n, const float* theta, int64_t ldt,
                                  int n_half, const int32_t* trans_host, int K, const float* G, void* dtheta,
                                  hipStream_t s);

// adj[cond[i]][b] += dx0[b][i]
hipError_t launch_scatter_add(float* adj, const float* dx0, int64_t n, int n_cond, const int32_t* cond_host,
                              hipStream_t s);

// G[b] = -F_b exp(-logq_b - logq_old_b) / n with F_b = wfj_b^2, and the loss
// sum_b F_b exp(...) / n into loss[0] (deterministic two-pass sum; `part`
// holds 1024 doubles).  log_loss: G is then divided by the loss (dlogL/dlogq).
hipError_t launch_flow_loss(int64_t n, const double* wfj, const float* logq, const float* logq_old, float* G,
                            double* part, double* loss, bool log_loss, hipStream_t s);

// Columns of the FP32 operands of the fused layers: lane l of the matrix
// instruction takes element 4 i + l / 16 of every 32 in its step i, so those
// eight stand together.
__host__ __device__ constexpr int32_t f32_operand_index(int32_t k) {
    return (k & ~31) | ((k & 3) << 3) | ((k >> 2) & 7);
}
// Where the operand copy of a layer orders its columns so: the offsets of W2,
// W3 and W4 and the end of W4 (0: nowhere).
struct OperandOrder {
    int32_t w2, w3, w4, end;
};
// Adam step on P parameters (bias corrections folded into lr_t, eps_t by the
// caller), then the operand copy of the parameters in `type`.  The copy pads
// each layer block of `per` parameters to `per_t` (a multiple of 8).
hipError_t launch_adam(int64_t P, float* params, const float* grad, float* m, float* v, float b1, float b2,
                       float lr_t, float eps_t, int type, void* params_t, int64_t per, int64_t per_t,
                       const OperandOrder& order, hipStream_t s);
hipError_t launch_cast(int64_t P, const float* params, int type, void* params_t, int64_t per, int64_t per_t,
                       const OperandOrder& order, hipStream_t s);

// u[k][i] = 24-bit Philox uniforms in (0, 1) (same counters as the FP64
// generator: key (seed, sid), counter (e0 + i, k / 4, 0, 0)).
hipError_t launch_uniform_f32(uint64_t seed, uint64_t sid, uint64_t e0, int64_t n, int d, float* u, hipStream_t s);

// y_d[k][i] = y[k][i] (FP32 -> FP64 for the mapping chain)
hipError_t launch_widen(int64_t count, const float* y, double* y_d, hipStream_t s);

// w[i] = wfj[i] * exp(logdet[i]); logq[i] = -logdet[i]
hipError_t launch_flow_weight(int64_t n, const double* wfj, const float* logdet, double* w, float* logq,
                              hipStream_t s);

}  // namespace msx
