// Host-side launch planning (declarations).  See grkan_walk.h for the walk the
// plan parameterises.
#ifndef GRKAN_PLAN_H_
#define GRKAN_PLAN_H_

#include "../../include/grkan.h"
#include "grkan_walk.h"

namespace grkan {

constexpr int kWavesPerWg = 4; // 256 threads per workgroup
constexpr int kThreadsPerWg = kWavesPerWg * kWave;

int elem_size(grkan_dtype_t io);
grkan_status_t check_shape(int64_t rows, int32_t D, int32_t G, grkan_dtype_t io);

// Fills the public plan and (optionally) the kernel-side walk parameters.
grkan_status_t make_plan(int64_t rows, int32_t D, int32_t G, grkan_dtype_t io, int32_t align_bytes,
                         int32_t num_cu, int32_t wg_per_cu, bool forward, grkan_plan_t *out, Walk *walk);

// The overlapped walk (grkan_walk.h) for groups that are not whole vectors: true if the shape takes it, with
// the plan and the walk.  It is an addition to make_plan, whose plans (and grkan_plan's) never overlap.
bool make_overlapped(int64_t rows, int32_t D, int32_t G, grkan_dtype_t io, int32_t num_cu, int32_t wg_per_cu,
                     bool forward, grkan_plan_t *out, Walk *walk);

// Rebuilds the walk parameters from a public plan (validating it).
grkan_status_t walk_from_plan(int64_t rows, int32_t D, int32_t G, grkan_dtype_t io,
                              const grkan_plan_t &pl, Walk *walk);

// Stage 2 of the backward pass (grkan_kernels.hip): adds `rows_per_group` workspace rows of m + 1 + n sums for each of the
// G groups into dA / dB, which it overwrites; coef says whether the numerator is shared and of which type they are.
struct CoefRows;
grkan_status_t run_stage2(const float *partial, int32_t rows_per_group, const CoefRows &coef, void *dA, void *dB, int32_t G,
                          int32_t m, int32_t n, struct ihipStream_t *stream);

// Coefficient sums whose second stage is still to run: rows_per_group workspace rows for each of G groups (degrees (5, 4)).
struct CoefSums;

// Parts of an MLP block's backward pass, all on bfloat16 tensors and parameters (arguments as grkan_bwd_model, grkan_hidden_bwd
// and grkan_linear_wgrad_pair have them, checked there); all but the last leave their second stage to it.  product_backward: the
// rational function's backward pass at x with dh W (W [K, N]) as the upstream gradient.
grkan_status_t bwd_model_stage1(const void *x, const void *dy, const CoefRows &coef, void *dx, void *dA, void *dB, grkan_alloc_t alloc,
                                void *alloc_context, int64_t rows, int32_t D, int32_t G, CoefSums *later, struct ihipStream_t *stream);
grkan_status_t hidden_bwd_stage1(const void *dout, const void *W, const void *h, const CoefRows &coef, void *dh, void *dA, void *dB,
                                 grkan_alloc_t alloc, void *alloc_context, int64_t rows, int32_t K, int32_t N, int32_t G, CoefSums *later,
                                 struct ihipStream_t *stream);
bool product_backward_pays(int64_t rows, int32_t K, int32_t N, int32_t G);
grkan_status_t product_backward(const void *dh, const void *W, const void *x, const CoefRows &coef, void *dx, void *dA, void *dB,
                                grkan_alloc_t alloc, void *alloc_context, int64_t rows, int32_t K, int32_t N, int32_t G, CoefSums *later,
                                struct ihipStream_t *stream);
grkan_status_t wgrad_pair_and_sums(const grkan_block_bwd_t &b, grkan_alloc_t alloc, void *alloc_context, const CoefSums (&sums)[2],
                                   struct ihipStream_t *stream);

} // namespace grkan
#endif // GRKAN_PLAN_H_
