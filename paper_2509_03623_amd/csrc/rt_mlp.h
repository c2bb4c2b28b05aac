// rt_mlp.h -- neural CO layer kernels (internal).
#pragma once
#include "../../include/rtcube.h"
#include "rt_kernels.h"

namespace rt {

// Prepared network: float biases per hidden layer, the output layer in float,
// the offsets of each layer in the flat float32 layout, the 16 Fourier
// frequencies, and the hidden layers in the kernels' element type, rows padded
// for LDS.
struct MlpDev {
    const float *b[4];
    const float *W5, *b5;
    int off[5];
    float freq[16];
    // the hidden layers as the A operand of the transposed product (output
    // neurons as rows); in BF16 the input order of layers 1..3 is permuted to
    // the accumulator layout of the layer before
    const void *Wr;
    // layers 1..3 transposed for the backward pass, [in][out], in BF16 with the
    // output order permuted like the accumulator packing
    const void *WrT;
};

size_t mlp_prep_bytes(int precision);
hipError_t mlp_prepare(const float *flat, int precision, void *buf, MlpDev *w, hipStream_t st);
// out is written at the points where the march reads the network
hipError_t mlp_forward(const Geometry &g, const Shade &s, const MlpDev &w, int precision, size_t M, float4 *out,
                       hipStream_t st);
// list: device scratch of mlp_backward_list_bytes (the list of the points with
// any dL/do != 0, with its chunks' counts; FP32: and the slabs)
size_t mlp_backward_list_bytes(size_t M, int precision);
hipError_t mlp_backward(const Geometry &g, const Shade &s, const MlpDev &w, int precision, size_t M,
                        const float4 *dO, uint32_t *list, float *dW, hipStream_t st);

} // namespace rt
