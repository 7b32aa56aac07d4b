// mlp.h -- layout constants and launch wrappers of the surrogate network.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lensed {

constexpr int MLP_IN = 17, MLP_H = 256, MLP_KPAD = 32;
// flat float32 parameters: W1 [256][17], b1, W2 [256][256], b2, W3 [256][256], b3, W4 [1][256], b4
constexpr int MLP_OFF_W1 = 0;
constexpr int MLP_OFF_B1 = MLP_OFF_W1 + MLP_H * MLP_IN;
constexpr int MLP_OFF_W2 = MLP_OFF_B1 + MLP_H;
constexpr int MLP_OFF_B2 = MLP_OFF_W2 + MLP_H * MLP_H;
constexpr int MLP_OFF_W3 = MLP_OFF_B2 + MLP_H;
constexpr int MLP_OFF_B3 = MLP_OFF_W3 + MLP_H * MLP_H;
constexpr int MLP_OFF_W4 = MLP_OFF_B3 + MLP_H;
constexpr int MLP_OFF_B4 = MLP_OFF_W4 + MLP_H;
constexpr int MLP_NPARAM = MLP_OFF_B4 + 1;
static_assert(MLP_NPARAM == 136449, "surrogate parameter count");
// bfloat16 weight copies: W1 padded to [256][32], W2, W3, W4, and (training) the
// transposes of W2 and W3
constexpr long MLP_WB_W2 = (long)MLP_H * MLP_KPAD;
constexpr long MLP_WB_W3 = MLP_WB_W2 + (long)MLP_H * MLP_H;
constexpr long MLP_WB_W4 = MLP_WB_W3 + (long)MLP_H * MLP_H;
constexpr long MLP_WB_W2T = MLP_WB_W4 + MLP_H;
constexpr long MLP_WB_W3T = MLP_WB_W2T + (long)MLP_H * MLP_H;
constexpr long MLP_WB_SIZE = MLP_WB_W3T + (long)MLP_H * MLP_H;

// Rows are processed 16, 32 or 64 to a block; buffers hold whole 64-row groups.
constexpr int MLP_ROW_GROUP = 64;
inline int mlp_padded_rows(int B) { return (B + MLP_ROW_GROUP - 1) / MLP_ROW_GROUP * MLP_ROW_GROUP; }
// Distance of two rows of a transposed buffer: off the powers of two, which would
// put the 64 rows a wave reads at once on few memory channels.
inline int mlp_transposed_stride(int rows) { return mlp_padded_rows(rows) + 64; }
constexpr int MLP_MAX_SPLITS = 32;   // parts the rows are split into for the weight gradients
constexpr int MLP_COLS = 4 * MLP_H;  // column sums of a row block: db1, db2, db3, dW4

// Device scratch for batches of at most `cap` rows (owned by the context; cap is
// a multiple of MLP_ROW_GROUP).
struct MlpScratch {
  int cap = 0;
  uint16_t* wb = nullptr;       // [MLP_WB_SIZE]
  uint16_t* X0T = nullptr;      // [32][cap + 64] normalised input, transposed
  uint16_t* HT[2] = {nullptr, nullptr};             // [256][cap + 64] activations of layers 1, 2, transposed
  uint16_t* dZT[3] = {nullptr, nullptr, nullptr};   // [256][cap + 64] back-propagated dZ, transposed
  float* d = nullptr;           // [cap]
  float* sq = nullptr;          // [cap]
  float* cols = nullptr;        // [cap / 16][MLP_COLS]
  float* dw = nullptr;          // [MLP_MAX_SPLITS][MLP_NPARAM]
};

// Adam: the factors of one update (host, float64, rounded once).
struct AdamStep {
  float lr, beta1, omb1, beta2, omb2, eps, bc1, bc2;
};
AdamStep adam_factors(int step, double lr, double beta1, double beta2, double eps);

hipError_t mlp_forward(const float* params, const float* norm, const float* x, float* y, int B, const MlpScratch& s,
                       hipStream_t st);
hipError_t mlp_grad(const float* params, const float* norm, const float* x, const float* yt, int B, float* grad,
                    float* loss, const MlpScratch& s, hipStream_t st);
hipError_t mlp_adam(float* params, const float* grad, float* m, float* v, int n, const AdamStep& a, hipStream_t st);
// mlp_grad and mlp_adam in one sequence; the gradient is not written.
hipError_t mlp_train(float* params, float* m, float* v, const AdamStep& a, const float* norm, const float* x,
                     const float* yt, int B, float* loss, const MlpScratch& s, hipStream_t st);

}  // namespace lensed
