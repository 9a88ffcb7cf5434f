// Entry points of the kernel files that the whole-step driver calls directly
// (below the argument checking of the C ABI), so that padded
// operands and scratch buffers are shared across the passes of one step.
#pragma once
#include <hip/hip_runtime.h>

#include <vector>

#include "../../include/rn50_hip.h"

namespace rn50 {

// The descriptor checks of the C ABI's own entry points (0, or the error code with the text set).
int conv_desc_check(const rn50_conv_desc* d, const char* who);
int bn_desc_check(const rn50_bn_desc* d, const char* who);

// conv.hip
size_t stem_padded_input_bytes(const rn50_conv_desc* d);
size_t stem_padded_weight_bytes(const rn50_conv_desc* d);
void stem_pad_input(const rn50_conv_desc* d, const void* x, void* xp, hipStream_t s);
// Batch-norm sums fused into a convolution's output stage come as one row of partial sums per output
// tile: `num` rows over `rows` consecutive output pixels each (the last row may cover fewer).
struct PartialRows {
  int rows, num;
};
PartialRows fwd_partial_rows(const rn50_conv_desc* d);    // tiles of the forward convolution's output
PartialRows dgrad_partial_rows(const rn50_conv_desc* d);  // tiles of the data gradient
int64_t dgrad_partial_rows_bound(const rn50_conv_desc* d);  // most rows any tile choice gives (tiles of >= 32 pixels)
// An inference-mode BN layer applied in a convolution's output stage: [relu](gamma*(product - mean)/sqrt(var + eps) +
// beta [+ residual]); residual: [M][Cout] or null.
struct BnAffine {
  const float *gamma, *beta, *mean, *var;
  float eps;
  int relu;
  const void* residual;
};
// bn_partial (null: none): the sums of the batch norm behind the convolution (bn_sums_at).
void stem_fwd_padded(const rn50_conv_desc* d, const void* xp, const void* w, void* wp, void* y, float* bn_partial,
                     hipStream_t s, const BnAffine* affine = nullptr);
// The BN sums that a convolution's output stage (or a stand-alone sums pass) leaves, one row per row tile.  Backward: the floats
// (sum g, sum g * xhat) per row and channel.  Forward, two forms: for a reader that adds rows up in every workgroup
// (bn_self_finalizes), the doubles (sum y, sum y^2), moved from the tile's shift to shift 0 by the writer so that the readers
// only add; else, for the finalize launch, the floats of a BnTileRow (shift, sums about it), which that launch moves to the
// first tile's shift in double: exact either way, and at 12544 rows the fewer bytes count.
// Eight channels by all rows are contiguous: the writer stores runs of 64 to 128 bytes (with the rows of a single channel
// contiguous its 2 to 3 * 64 sums were a partial cache line each), and a finalize workgroup reads one run of memory
// (row-major, it picked 64 bytes out of every row: 12544 rows, batch 256, 45 us).
__host__ __device__ inline int64_t bn_sums_at(int row, int c, int nrows) {
  return (static_cast<int64_t>(c >> 3) * nrows + row) * 8 + (c & 7);
}
// Bytes per row and channel; bn_sums_bytes: of nrows rows.
constexpr int kBnBwdSumBytes = 8, kBnTileRowBytes = 12, kBnWideSumBytes = 16;
inline size_t bn_sums_bytes(int64_t nrows, int C, int each) { return static_cast<size_t>(nrows) * ((C + 7) / 8 * 8) * each; }
// They are added up by a finalize launch, or, when there are few tile rows, by the BN apply pass (forward or backward)
// itself, in every workgroup, for the channels it applies: the launch in front of it -- about 4 us on the step's
// dependency chain whatever it computes -- is gone.
// Threshold from whole-step measurements (profiles/step_time_against_dispatch_constants.txt; batch 40, 64 / 128 / 256 / 512 rows
// against none: 4.234 / 4.234 / 4.328 / 4.328 against 4.250 ms): up to 123 tile rows (the 14x14 and 7x7 layers) the
// redundant sums cost less than the launch; at 245 (28x28) every workgroup would read more sums than data.  (At batch 256 256
// rows are 0.2 % slower, 512 0.7 %.)
constexpr int kBnSelfFinalizeRows = 128, kBnSelfFinalizeRowsBwd = 128;
inline bool bn_self_finalizes(int nrows, bool backward) {
  return nrows <= (backward ? kBnSelfFinalizeRowsBwd : kBnSelfFinalizeRows);
}

// More tile rows than a finalize launch should read: the producer adds them up, in double, to kBnReducedRows rows of doubles
// behind its own (bn_reduced_rows; there is room: such a layer's tiles have at least 64 pixels, the buffer is sized for tiles
// of 32), and the finalize launch reads these.  Why and where the line lies: bn_reduce_rows_kernel.
constexpr int kBnReduceRows = 4096, kBnReducedRows = 64;
inline bool bn_reduces(int nrows) { return nrows > kBnReduceRows; }
inline double2* bn_reduced_rows(const float* sums, int nrows, int C, bool backward) {
  const size_t own = bn_sums_bytes(nrows, C, backward ? kBnBwdSumBytes : kBnTileRowBytes);  // (a multiple of 32)
  return reinterpret_cast<double2*>(reinterpret_cast<uintptr_t>(sums) + own);
}
// bn.hip.  rpp: rows of x behind a row of sums (forward), m: of x in all.
void bn_reduce_rows(float* sums, int nrows, int rpp, int64_t m, int C, bool backward, hipStream_t s);

// An apply pass whose launch also finalizes (kFinShared): one word per channel, made empty by the producer of the sums, and how
// often a workgroup asks for another one's results before it computes them itself.
constexpr unsigned long long kBnSlotEmpty = ~0ull;
constexpr int kBnPolls = 2000;
struct BnShare {
  unsigned long long* slots;
  int polls;
};
// Sets `polls` for a plan's steps (0: every workgroup computes what it needs itself).  Not part of the library's interface: no
// value of it is of use to a caller.  The tests show with it that the results are the same whoever computed them.
extern "C" int rn50_internal_wait_polls(rn50_plan* plan, int polls);

// A BN+ReLU layer applied to a convolution's input on the fly (1x1, stride 1 convolutions only): its parameters
// and saved statistics, float[Cin] each.
struct BnIn {
  const float *gamma, *beta, *mean, *rstd;
};
void fwd_run(const rn50_conv_desc* d, const void* x, const void* w, void* y, float* bn_partial, hipStream_t s,
             const char* tag = "conv_fwd", const BnIn* in = nullptr, const BnAffine* affine = nullptr,
             unsigned long long* slots = nullptr);  // slots: to be made empty (BnShare)
// The BN layer (with ReLU) whose output gradient a data gradient produces: x is that
// layer's input [N*H*W][Cin]; partial receives the pairs sum(g), sum(g * xhat) per tile and channel (bn_sums_at).
// addend (or null): a second branch of the gradient, [N*H*W][Cin], added to the data gradient before it
// is stored; relu_mask (or null): the BN layer's recorded ReLU decisions (else recomputed from x);
// addend_mask (or null): ReLU bits under which the addend counts (the addend is then the still unmasked
// output gradient of the residual-add layer that recorded them).
struct BnBwdSums {
  const void* x;
  const float *gamma, *beta, *mean, *rstd;
  float* partial;
  const void* addend = nullptr;
  const uint8_t* relu_mask = nullptr;
  const uint8_t* addend_mask = nullptr;
  unsigned long long* slots = nullptr;  // to be made empty (BnShare)
  bool addend_even = false;  // the addend's pixels with odd row or column are zero and left out (1x1 / stride 1, no addend_mask)
};
void dgrad_run(const rn50_conv_desc* d, const void* dy, const void* w, void* dx, const BnBwdSums* bn, hipStream_t s,
               const char* tag = "conv_dgrad");
size_t wgrad_partial_bytes(const rn50_conv_desc* d);
void wgrad_run(const rn50_conv_desc* d, const void* x_or_xp, const void* dy, float* dw, void* scratch, hipStream_t s,
               const BnIn* in = nullptr);

// bn.hip.  last_reader: the operands are not read again for a long while (bn_apply_kernel's LAST).
// The part of the forward / backward pass that follows the sums.
void bn_fwd_from_partials(const rn50_bn_desc* d, const void* x, const float* partial, int nrows, int rpp,
                          const float* gamma, const float* beta, const void* residual, void* y,
                          uint8_t* relu_mask, float* save_mean, float* save_rstd, float* rm, float* rv,
                          float momentum, bool last_reader, hipStream_t s, const BnShare* share = nullptr);
// relu_mask: recorded ReLU decisions (required in mode 2, where dres receives the masked gradient), or
// null: recomputed from x (mode 1).
void bn_bwd_from_partials(const rn50_bn_desc* d, const void* dz, const void* x, const uint8_t* relu_mask,
                          const float* gamma, const float* beta, const float* mean, const float* rstd,
                          const float* partial, int nrows, void* dx, void* dres, float* dgamma, float* dbeta,
                          bool last_reader, hipStream_t s, const BnShare* share = nullptr);
// The whole backward pass (bn_relu_bwd without its checks); scratch: bn_relu_bwd_workspace_bytes(d).
void bn_bwd_run(const rn50_bn_desc* d, const void* dz, const void* dz2, const void* x, const void* z,
                const uint8_t* relu_mask, const float* gamma, const float* beta, const float* mean, const float* rstd,
                void* dx, void* dres, float* dgamma, float* dbeta, float* scratch, bool last_reader, hipStream_t s);
// relu(bn(x)) of known statistics, through the 3x3 / stride 2 / padding 1 max-pool: pooled output and winners (maxpool_fwd's)
// from the BN layer's input.
void bn_relu_maxpool(const rn50_bn_desc* d, const void* x, const float* gamma, const float* beta, const float* mean,
                     const float* rstd, void* pooled, uint8_t* argmax, hipStream_t s);

// head.hip: the pieces of xent_fwd_bwd and fc_bwd that a step runs on different streams.
// The rows of the loss: row_loss, dlogits and (bf16, or null) the copy of dlogits rounded to the storage type.
void xent_rows(int N, int K, const float* logits, const int32_t* labels, float label_smoothing, float grad_scale,
               float* row_loss, float* dlogits, void* dlogits_t, int dtype, hipStream_t s);
void loss_mean(int N, const float* row_loss, float* loss_out, hipStream_t s);
// The classifier's data gradient from dlogits in the storage type (Cin and K multiples of the 16-byte vector).
bool fc_mfma_ok(int Cin, int K, int dtype);
void fc_bwd_da(int N, int Cin, int K, int dtype, const void* W, const void* dlogits_t, void* da, hipStream_t s);
// The classifier's parameter gradients alone (fc_bwd with dW = db = null leaves them out).
void fc_bwd_params(int N, int Cin, int K, int dtype, const void* a, const float* dlogits, float* dW, float* db,
                   hipStream_t s);

// lars.hip
struct LarsArenaSpec {
  int num = 0;
  std::vector<int64_t> offset, count;
  std::vector<char> decay;
};
size_t lars_arena_partial_bytes(const LarsArenaSpec& sp);
void lars_arena_run(const LarsArenaSpec& sp, float* master, const float* grads, float* velocity, void* lowp,
                    float eta, float momentum, float lr, const float* lr_dev, float eps, float weight_decay,
                    float* partial, int64_t arena_elems, hipStream_t s);

}  // namespace rn50
