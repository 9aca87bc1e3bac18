// Host-callable launchers of the HIP kernels (one translation unit each).
#pragma once
#include "common.hpp"

namespace qasr {

// Generic direct convolution: any stride / dilation / padding / channel count, dense or
// depthwise.  One thread per output element.  The fallback for geometries the MFMA kernels
// do not take.
hipError_t launch_conv_generic(const ConvParams& p, hipStream_t st);

// Standalone epilogue on int32 accumulators.
hipError_t launch_requant(const int32_t* acc, int B, int C, int T, const int32_t* bias,
                          const int32_t* m, const int32_t* s, const int8_t* res, int relu,
                          int8_t* y, hipStream_t st);

// [Cout][Cin][k] -> MFMA operand order (common.hpp: packed_weight_index); needs Cin % 64 == 0
hipError_t launch_pack_weights(const int8_t* w, int8_t* wp, int Cout, int Cin, int k, hipStream_t st);

// Depthwise convolution as a banded-Toeplitz product on the int8 matrix cores (stride 1).
bool dw_mfma_supported(const ConvParams& p);
hipError_t launch_dw_mfma(const ConvParams& p, hipStream_t st);

// Pointwise / dense convolution as an implicit GEMM on the int8 matrix cores.
bool gemm_mfma_supported(const ConvParams& p);
hipError_t launch_gemm_mfma(const ConvParams& p, hipStream_t st);

// Depthwise convolution, same arithmetic, software-pipelined over the batch (reads and writes of
// HBM overlap); needs aligned rows, no residual and enough rows per wave to pipeline.
bool dw_pipe_supported(const ConvParams& p);
hipError_t launch_dw_pipe(const ConvParams& p, hipStream_t st);

// Pointwise convolution (k = 1), activation tile stationary in LDS (direct global->LDS loads);
// needs packed weights, rows that are a multiple of 16 frames and Cin <= 1024.
bool pw_tile_supported(const ConvParams& p);
hipError_t launch_pw_tile(const ConvParams& p, hipStream_t st);

// Pointwise convolution (k = 1), activation tile stationary in LDS, output channels in passes of
// 256 whose epilogues run in between the matrix products of the following pass; needs packed
// weights, rows that are a multiple of 16 frames, Cin in {256, 512} and 256 <= Cout <= 2048.
bool pw_pipe_supported(const ConvParams& p);
hipError_t launch_pw_pipe(const ConvParams& p, hipStream_t st);

// Pointwise convolution (k = 1), 16 waves per workgroup, the whole tile in flight at once; packed weights,
// Cin a multiple of 64 up to 2048, rows of any length.  pw_wide_better: whether it is the faster choice for
// a layer that pw_pipe (pipe) or pw_tile takes.
bool pw_wide_supported(const ConvParams& p);
bool pw_wide_better(const ConvParams& p, bool pipe);
hipError_t launch_pw_wide(const ConvParams& p, hipStream_t st);
// its model of a layer's time on the whole chip, us without the launch; false where it does not take the layer
bool pw_wide_us(const ConvParams& p, double& us);
// Several pointwise layers of equal output shape, none of which reads what another writes, in one launch of pw_wide's
// tiles; pw_multi_better: whether they can and it is the faster way.
constexpr int kMaxMulti = 12;
bool pw_multi_better(const ConvParams* p, int n);
hipError_t launch_pw_multi(const ConvParams* p, int n, hipStream_t st);

// Dense convolution (k >= 2) as an implicit GEMM pipelined over (chunk, tap) steps; needs packed
// weights, Cin % 64 == 0, Cout >= 64.
bool conv_pipe_supported(const ConvParams& p);
// Bytes of ConvParams::part with which the layer's launch would split its contraction over several
// workgroups per tile, 0 if it would not; the counters beside it are zero before and after each launch.
constexpr int kConvSplitCounters = 1024;
size_t conv_pipe_split_bytes(const ConvParams& p);
hipError_t launch_conv_split_clear(unsigned* counters, hipStream_t st);
hipError_t launch_conv_pipe(const ConvParams& p, hipStream_t st);

// The same layers in launches of few frames: all input channels of a small tile in LDS, the weights streamed by 16
// free-running waves, no workspace.  A tile is MT groups of 16 frames and WC column waves of NT 16-channel columns each.
// conv_few_cycles: the fastest tile and its estimate, on conv_pipe's scale; conv_few_better: whether that is the faster
// choice for a layer that conv_pipe takes (split: there is a workspace for that to split its contraction).  A launch takes the
// tile that was chosen, for the layer and for the next one: models are evaluated once per layer and forward.
struct FewTile { int MT, WC, NT; };
bool conv_few_cycles(const ConvParams& p, FewTile& tile, double& cycles);
bool conv_few_better(const ConvParams& p, bool split, FewTile& tile);
// next: the next layer that this kernel will run, with its tile (or null), whose weights are brought into the L2s meanwhile
hipError_t launch_conv_few(const ConvParams& p, const FewTile& tile, const ConvParams* next, const FewTile& next_tile, hipStream_t st);

// Measured ceilings (probe.hip): a streaming copy of `bytes` (a multiple of 16) and a register-resident
// int8 matrix-core loop of probe_mfma_ops(iters) operations that writes probe_mfma_workgroups() int32.
hipError_t launch_probe_copy(const void* src, void* dst, size_t bytes, hipStream_t st);
int probe_mfma_workgroups();
double probe_mfma_ops(int iters);
hipError_t launch_probe_mfma(int iters, int32_t* out, hipStream_t st);

// Quantiser (Eq. 1, b = 8; S = alpha / 127 from the host) and dequantiser (S * q) at the two ends
// of the path; n elements, any alignment.
hipError_t launch_quantize(const float* x, size_t n, float alpha, float S, int8_t* q, hipStream_t st);
hipError_t launch_dequantize(const int8_t* q, size_t n, float S, float* x, hipStream_t st);
// The same between dense float rows of T frames and int8 rows of `pitch` >= T bytes (a multiple of 4,
// 4-byte aligned).
hipError_t launch_quantize_rows(const float* x, int64_t rows, int T, float alpha, float S, int8_t* q, int pitch, hipStream_t st);
hipError_t launch_dequantize_rows(const int8_t* q, int64_t rows, int T, int pitch, float S, float* x, hipStream_t st);

// Integer-only activations (Sec. 2.2: second-order polynomial exponential).  kind 1 sigmoid,
// 2 swish, 3 GLU; u refines an int8 code to scale S / 2^u; q_ln2, q_b, q_c are the host-side
// constants of the exponential at that scale; (m, s) the dyadic rescale of the result.
struct ActParams {
  int32_t kind, m, s, u;
  int64_t q_ln2, q_b, q_c;
};
// table[code + 128] = int8 output of the unary activation (sigmoid, swish) for every int8 code
hipError_t launch_act_table(const ActParams& c, uint8_t* table, hipStream_t st);
// table[code + 128] = 16-bit sigmoid code of a GLU's gate, for every int8 code
hipError_t launch_glu_table(const ActParams& c, uint16_t* table, hipStream_t st);
// x: B items of n (2 n for GLU: value half, gate half) int8 at stride xbs; y: B items of n int8
// at stride ybs; y may be x itself when the strides are equal.
hipError_t launch_act(const ActParams& c, const int8_t* x, int8_t* y, int32_t B, int64_t n, int64_t xbs,
                      int64_t ybs, hipStream_t st);
// rows x L int32 logits -> int8 probabilities at scale 2^-7 (kind, m, s unused).
hipError_t launch_softmax(const ActParams& c, const int32_t* x, int64_t rows, int32_t L, int8_t* y, hipStream_t st);

// Offline calibration helpers (Sec. 2.1, 2.2, 3.1): running (min, max) of float32 values into
// mm[0..1] (device); the dyadic form of a positive multiplier (host or device arithmetic, the
// same function); BatchNorm folding + per-channel weight quantisation + bias and (m, s).
hipError_t launch_minmax(const float* x, size_t n, float* mm, hipStream_t st);
bool dyadic_from_scale(double M, int32_t& m, int32_t& s);
hipError_t launch_fold_quantize(const float* w, const float* b, const float* gamma, const float* beta, const float* mean,
                                const float* var, float eps, int32_t Cout, int64_t per, float S_x, float S_y, int8_t* qw,
                                int32_t* bias_q, int32_t* m, int32_t* s, float* S_w, int32_t* bad_count, hipStream_t st);

}  // namespace qasr
