// What the direct method's dispatch (direct_mfma.hip) needs of the kernel on split operands (direct_split.hip).
#pragma once

#include "znn_internal.h"

namespace znn {

struct SplitChoice {
    bool ok;
    int NJ, jgroups, NV, NW;        // 16-map tiles per workgroup, groups of them, 16-voxel tiles per wave, waves
    int T[3], H[3], c[3];           // box, halo box, boxes per sublattice (z, y, x)
    int phases, steps, nchunk;
    int cps, splits;                // chunks of eight input maps per workgroup, shares of them
    size_t lds;
    double cost;                    // expected clocks
};

SplitChoice choose_split(const Geom& g, bool backward);      // ok = false: the fp32 kernel takes the pass
size_t split_packed_bytes(const SplitChoice& c);
int split_conv(const Geom& g, bool backward, const float* src, const void* wp, float* dst, float* partial, const Finish& finish,
               hipStream_t s);

}  // namespace znn
