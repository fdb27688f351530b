// The backward pass of an MLP block as one call: four launches where each rational function runs inside the product beside it, one more for
// each that does not, where the rows of a product are split (grkan_product_tile), or where the weight gradients take a launch each;
// the parts by themselves take three more (their second stages, and the sums of the weight gradients).
#include <hip/hip_runtime.h>

#include "grkan_elem.h"
#include "grkan_plan.h"

using namespace grkan;

extern "C" grkan_status_t grkan_block_bwd(const grkan_block_bwd_t *b, grkan_alloc_t alloc, void *alloc_context, void *hip_stream)
{
    if (!b || !alloc)
        return GRKAN_ERR_NULL;
    if (b->rows <= 0 || b->D <= 0 || b->hidden <= 0)
        return GRKAN_ERR_SHAPE;
    if (!grkan_hidden_supported(b->D, b->hidden, b->G2) || !grkan_product_supported(b->rows, b->hidden, b->D))
        return GRKAN_ERR_UNSUPPORTED;
    if (!b->dh)
        return GRKAN_ERR_NULL;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const CoefRows c1{b->A1, b->B1, b->shared1 ? 0 : 6, 1}, c2{b->A2, b->B2, b->shared2 ? 0 : 6, 1};
    CoefSums sums[2];
    grkan_status_t st;
    if (grkan_hidden_pays(b->rows, b->D, b->hidden, b->G2, 1)) {
        st = hidden_bwd_stage1(b->dout, b->W2, b->h, c2, b->dh, b->dA2, b->dB2, alloc, alloc_context, b->rows, b->D, b->hidden, b->G2, &sums[1],
                               stream);
    } else {
        // (dF2, the largest tensor of the pass, is dh's memory until F2's backward pass writes dh over it, element by element)
        st = grkan_product(b->dout, b->W2, nullptr, b->dh, b->rows, b->D, b->hidden, 1, nullptr, nullptr, 1, 0, hip_stream);
        if (st == GRKAN_OK)
            st = bwd_model_stage1(b->h, b->dh, c2, b->dh, b->dA2, b->dB2, alloc, alloc_context, b->rows, b->hidden, b->G2, &sums[1], stream);
    }
    if (st == GRKAN_OK && product_backward_pays(b->rows, b->hidden, b->D, b->G1)) {
        st = product_backward(b->dh, b->W1, b->x, c1, b->dx, b->dA1, b->dB1, alloc, alloc_context, b->rows, b->hidden, b->D, b->G1, &sums[0],
                              stream);
    } else if (st == GRKAN_OK) {
        void *const df1 = alloc((size_t)b->rows * (size_t)b->D * 2, alloc_context);
        if (!df1)
            return GRKAN_ERR_WORKSPACE;
        st = grkan_product(b->dh, b->W1, nullptr, df1, b->rows, b->hidden, b->D, 1, nullptr, nullptr, 1, 0, hip_stream);
        if (st == GRKAN_OK)
            st = bwd_model_stage1(b->x, df1, c1, b->dx, b->dA1, b->dB1, alloc, alloc_context, b->rows, b->D, b->G1, &sums[0], stream);
    }
    return st == GRKAN_OK ? wgrad_pair_and_sums(*b, alloc, alloc_context, sums, stream) : st;
}
