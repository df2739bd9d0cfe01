// Argument blocks of the grouped launches: several layers of one shape whose upstream gradients
// do not depend on each other (the Q, K and V projections of an attention block) run each step of
// the path in ONE launch, blockIdx.y (blockIdx.x for the one-workgroup samplers) picking the layer.
// Every layer is computed by the code of the single-layer kernel, so its bits do not change.
#pragma once

#include "rowsum.hpp"
#include "sample_a_small.hpp"

namespace vcas {

constexpr int kMaxSiblings = 4;
constexpr int kMaxSamplers = 8;   // samplers in one launch: siblings, or mask draws of the variance probe

// One layer of a grouped dgrad launch (layers of one shape that do not depend on each other):
// the pointer arguments of the bf16 dgrad kernel.
struct DgradProblem {
    const uint16_t *G, *W;
    const float *p;
    const int32_t *idxA, *cntA;
    uint16_t *dX;
    const uint16_t *J;   // null: no Jacobian
    InlineSampleA sa;    // sa.gsq null: SampleA has been decided, p / idxA / cntA hold its outcome
    float *sq_blocks;    // null, or the sums of squares of the written dX by blocks of 64 columns (layout: rows_from_blocks)
};
struct DgradGroup {
    DgradProblem prob[kMaxSiblings];
};

// SampleA of several layers in one launch: one workgroup each, the fields of InlineSampleA.
struct SampleAGroup {
    InlineSampleA prob[kMaxSamplers];
};

// One layer of a batched bf16 weight-gradient launch (host view): the arguments of
// vcas_sampled_wgrad, where its split-K partial tiles and its packed (gathered and pre-scaled)
// narrower operand go, and how many slices its contraction is cut into.
constexpr int kWgradBatch = 8;
struct WgradItem {
    vcas_shape shape;
    const void *G, *X;
    const float *row_scale;
    const int32_t *idxW, *cntW;
    float *dW, *partials;
    uint16_t *packed;
    int splits;
};

// One layer of a grouped SampleW launch: the pointer arguments of the one-workgroup sampler.
struct SampleWProblem {
    float *xsq;
    const float *p;
    const uint8_t *maskA;
    float *u;       // uniforms by row; a long vector's counts lie over them once they have been compared
    double budget;
    float *score, *q;
    uint8_t *maskW;
    float *scaleW;
    int32_t *idxW, *cntW;
    double *rule;   // [2], scratch of the workspace: the keep rule of a long vector
};
struct SampleWGroup {
    SampleWProblem prob[kMaxSamplers];
};

// The same for the row-norm launch: matrix, where its row sums go, and (null: all) the samples
// whose rows are read at all.
struct RowNormGroup {
    const uint4 *A[kMaxSiblings];
    float *out[kMaxSiblings];
    const uint8_t *keep[kMaxSiblings];
};

// Row norms with their side jobs (SampleW's scores and uniforms) for up to kMaxSamplers matrices of one shape
// in one launch.  Where norms is set, the sums of squares of every row are read there and the matrix is not.
struct RowJobGroup {
    const uint4 *A[kMaxSamplers];
    const float *norms[kMaxSamplers];
    const uint8_t *keep[kMaxSamplers];
    float *out[kMaxSamplers];
    UniformJob job[kMaxSamplers];
    ScoreJob sj[kMaxSamplers];
};

}  // namespace vcas
