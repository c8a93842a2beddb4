// Launch interface of the training kernels of the float (sigmoid) networks:
// the mean softmax cross-entropy of the logits against the labels and its
// gradient by backpropagation (the networks are trained on labelled
// examples, Sec. II-A; the verifier's counterexamples are added to the
// training set, Sec. VI).
#pragma once

#include "ibmc_internal.h"

namespace ibmc {

constexpr int kTrainTile = 4;              // samples per workgroup of the pass
constexpr int kTrainMaxGroup = 16;         // samples per running sum (train_group)

// The flat parameter vector theta: for each layer l = 1..L in turn, W_l
// row-major [dims[l]][dims[l-1]] then b_l [dims[l]].
struct TrainNetDev {
    int L;
    int dims[kMaxLayers + 1];
    int64_t toff[kMaxLayers + 1];   // l >= 1: offset of W_l in theta (b_l follows it)
    int64_t n_params;
    // per-sample row of activations a_0 .. a_L (a_L = the logits) at aoff[l],
    // each layer padded to four; deltas dL/du of layers 1..L in the same places
    int aoff[kMaxLayers + 1];
    int units;
    int widest;                     // widest layer, padded to four
};

TrainNetDev train_layout(int L, const int *dims);

// Samples per running sum: a gradient entry is the sum, in sample order, of
// the sums over groups of this many samples (and so is the loss).  At most
// `wanted`, and fewer for wide networks.  Part of the results' definition:
// another group rounds otherwise.
int train_group(const TrainNetDev &N, int wanted);

// One pass over elements e0 .. e0 + count - 1: rows of activations and deltas
// (count padded to kTrainTile rows) and each sample's loss.
struct TrainPassParams {
    TrainNetDev net;
    const float *theta;
    const uint8_t *images;     // [n_images][dims[0]]
    const int32_t *labels;     // [n_images], each in [0, dims[L])
    const int64_t *order;      // nullable: element e of the pass is image order[e]
    int64_t e0, count;
    float inv_n;               // 1 / the number of samples the mean runs over
    float *acts, *dels;        // [rows][units]
    float *loss;               // [count]
    int group;                 // samples per running sum
};

// What becomes of the weight gradients of a pass.
struct TrainUpdate {
    float *grad;               // non-null: grad = (accumulate ? grad : 0) + gradient
    int accumulate;
    float *theta, *mom, *vel;  // grad null: one Adam step
    float lr, b1, b2, eps, c1, c2;
    double *loss_acc;          // += the pass's loss sum
};

hipError_t launch_train_pass(const TrainPassParams &P, hipStream_t s);
hipError_t launch_train_weights(const TrainPassParams &P, const TrainUpdate &U, hipStream_t s);

}  // namespace ibmc
