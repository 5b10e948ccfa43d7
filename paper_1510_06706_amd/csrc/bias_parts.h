// Sums of the bias gradients of a round: one workgroup per map and kBiasSpan voxels, of any of its layers.
#pragma once

#include "znn_internal.h"

namespace znn {

constexpr int kBiasSpan = 8192;
struct BiasItem { const float* g; float* parts; long voxels; int spans; unsigned first; };     // first: workgroup it starts at

// red: four floats of LDS; workgroups of 256 threads
__device__ __forceinline__ void bias_part(const BiasItem& B, unsigned r, float* red)
{
    const unsigned m = r / B.spans, span = r % B.spans;
    const float* p = B.g + (long)m * B.voxels + (long)span * kBiasSpan;
    const int n = (int)min((long)kBiasSpan, B.voxels - (long)span * kBiasSpan);
    float a[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) a[i] = 0.f;
    for (int t = threadIdx.x; t < n; t += 2048)
#pragma unroll
        for (int i = 0; i < 8; ++i) a[i] += t + i * 256 < n ? p[t + i * 256] : 0.f;
    float v = ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
    for (int s = 32; s > 0; s >>= 1) v += __shfl_down(v, s);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) B.parts[r] = (red[0] + red[1]) + (red[2] + red[3]);
}

// Kernel gradients of several layers on the vector ALUs (grad_is_few) and, beside them, the sums of biases: launches by the widths of their
// groups of taps, the biases (at most kFewBiases of them in kFewBiasGroups workgroups, `first` counted from zero) with the first one.
constexpr int kFewBiases = 24;
constexpr unsigned kFewBiasGroups = 1u << 16;
int few_grads(const GradItem* items, int count, const BiasItem* bias, int biases, unsigned bias_groups, hipStream_t s);

}  // namespace znn
