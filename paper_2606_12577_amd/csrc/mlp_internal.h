// Internal declarations of the block-smoother network (learned setup).
#pragma once

#include <functional>

#include "cs_internal.h"
#include "../../include/cascade_learned.h"

namespace cs {

struct Mlp {
    int device = 0;
    hipStream_t stream = nullptr;
    std::string err;
    int n_in = 0, width = 0, n_out = 0;
    int64_t np = 0;                       // parameter count
    int64_t off[7] = {0};                 // W1, b1, W2, b2, W3, b3, end
    DBuf<float> p, g, m, v;               // parameters, gradient, Adam moments
    DBuf<float> mean, std;                // output scaling
    int64_t step = 0;                     // Adam steps taken
    // activations of one batch (capacity rows)
    int64_t cap = 0;
    DBuf<float> z1, h1, z2, h2, y, dy, d2, d1;
    DBuf<double> part, acc;               // loss partial sums
    DBuf<float> kpart;                    // split-k partial products
    // row-tile path (mlp_rows.hip): first-layer products, activations and
    // deltas [rows][128], partial gradients, loss partial sums
    DBuf<float> r_part, r_h1, r_h2, r_dy, r_d2, r_d1, r_wpart, r_bpart;
    DBuf<double> r_lpart;
    double *h_acc = nullptr;              // pinned readback
    size_t h_acc_cap = 0;
};

// Y = prediction in target units for n rows of X (on stream s)
void mlp_predict(Mlp &m, hipStream_t s, const float *X, int64_t n, float *Y);

// mlp_rows.hip: networks of hidden and output widths of at most 128
struct AdamRate {
    float lr, b1, b2, eps, c1, c2;   // c1, c2: the moments' bias corrections
};
bool rows_path(const Mlp &m, const float *X);
void rows_predict(Mlp &m, hipStream_t s, const float *X, int64_t n, float *Y);
void rows_loss(Mlp &m, hipStream_t s, const float *X, const float *T, const int32_t *rows, int64_t n);
void rows_gradient(Mlp &m, hipStream_t s, const float *X, const float *T, const int32_t *rows, int64_t n);
void rows_epoch(Mlp &m, hipStream_t s, const float *X, const float *T, const int32_t *order, int64_t n_train,
                int64_t batch, const std::function<AdamRate()> &rate);

}  // namespace cs

struct cs_mlp_s {
    cs::Mlp m;
};
