// gc_mlp_launch.h -- host-side launchers of the neural-field kernels.
#pragma once
#include <hip/hip_runtime.h>

#include "gc_internal.h"
#include "gc_mlp.h"

namespace gc {

struct MlpLoss {
    double wc[kMlpOut];   // weights of the six normalized outputs
    double beta;          // weight of the paired-difference term
};

// Parameters of the network on the device: FP32 masters p with their gradient
// and Adam moments, c, co and Wo_master within p, and the BF16 copies.
struct TrainNet {
    float *p, *mo, *ve, *g;
    const float *c, *co, *Wo_master;
    __bf16 *W, *WT, *Wo, *We, *Woe;
};
struct AdamArgs {
    float lr, b1, b2, eps, c1, c2;   // c1 = 1 - b1^step, c2 = 1 - b2^step
    int apply;                       // 0: gradient only
};
// Workspace of a training step
struct TrainBufs {
    float *Y;             // outputs [rows][6]
    __bf16 *HT, *DT;      // transposed tiles of H_0..H_5 and of dZ_1..dZ_6
    float *part;          // weight-gradient chains [6][4][128][128]
    float *sums;          // per block: bias gradients, dWo, dco
    double *loss;         // per block
};
constexpr int kTrainRows = 64;                                      // of a block
constexpr int kTrainSums = kMlpDepth * kMlpWidth + kMlpOut * kMlpWidth + kMlpOut;
__host__ __device__ constexpr int mlp_train_blocks(int64_t npair) {
    return (int)((2 * npair + kTrainRows - 1) / kTrainRows);
}
// Rows of a weight-gradient group: about 128 groups, of whole 16-row products and
// at least 128 rows.
__host__ __device__ constexpr int mlp_train_chunk(int rows) {
    const int g = rows / 128 < 1 ? 1 : rows / 128 > 128 ? 128 : rows / 128;
    return ((rows + g - 1) / g + 15) / 16 * 16;
}
// One training step.  *loss_host (coherent host memory) receives the loss.
hipError_t mlp_launch_train(const MlpArgs &m, const TrainNet &net, const double *pts, const double *tgt, int npair,
                            const MlpLoss &L, const AdamArgs &adam, const TrainBufs &w, volatile double *loss_host,
                            hipStream_t s);
hipError_t mlp_launch_refresh(const float *p, __bf16 *W, __bf16 *WT, __bf16 *Wo, __bf16 *We, __bf16 *Woe,
                              hipStream_t s);
hipError_t mlp_launch_eval(const MlpArgs &m, const double *pts, int n, double *out, int cus, hipStream_t s);
hipError_t launch_field_sample(const FieldDev &f, const double *pts, int n, double *out, hipStream_t s);
hipError_t launch_push_mlp(const PushArgs &a, const MlpArgs &m, int precision, int cus, hipStream_t s);

}  // namespace gc
