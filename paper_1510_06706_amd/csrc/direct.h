// The kernels of the direct method, as its dispatch (direct.hip) sees them.
#pragma once

#include <type_traits>

#include "znn_internal.h"

namespace znn {

// ---- forward and backward pass on split operands (direct_split.hip)
struct SplitChoice {
    bool ok;
    int NJ, jgroups, NV, NW;        // 16-map tiles per workgroup, groups of them, 16-voxel tiles per wave, waves
    int T[3], H[3], c[3];           // box, halo box, boxes per sublattice (z, y, x)
    int phases, steps, nchunk;
    int cps, splits;                // chunks of eight input maps per workgroup, shares of them
    bool beside;                    // four more waves stage beside those that multiply (direct_beside_impl.h), else these in between (direct_split_impl.h)
    int hop, wofs, whop, tables;    // beside, LDS: from one staging buffer to the other (0: one buffer), weights and their second buffer, tables
    size_t lds;
    double cost, between;           // expected clocks, and those of the best choice whose waves stage in between
    int boxes;                      // that the search looked at
};
SplitChoice choose_split(const Geom& g, bool backward);
bool split_place(SplitChoice& c);
double split_seconds(double clocks);
size_t split_packed_bytes(const SplitChoice& c);
PackItem split_pack_item(const Geom& g, const SplitChoice& c, bool backward, const float* w, void* wp);
int split_pack_weights(const PackItem* items, int n, hipStream_t s);
// `shares` shares of the input maps from share0 on, 0: all of them.  More than one: a result array of `partial` each; one: into dst.
int split_conv(const Geom& g, const SplitChoice& c, bool backward, const float* src, const float* w, const void* wp, float* dst, float* partial,
               const Finish& finish, hipStream_t s, int share0 = 0, int shares = 0);

// ---- kernel gradient on split operands (direct_wgrad_split.hip)
bool split_grad_supported(const Geom& g);
double split_grad_seconds(const Geom& g);
size_t split_grad_sums_bytes(const Geom& g);
size_t split_grad_copies_bytes(const Geom& g);
int split_grad(const Geom& g, const GradItem& item, hipStream_t s);
bool split_grad_joins(const Geom& g);
int split_grads(const GradItem* items, int count, hipStream_t s);
int sum_shares(const WgradSum& S, const float* partial, float* gw, hipStream_t s);

// ---- all passes on the vector ALUs (direct_few.hip)
double few_conv_seconds(const Geom& g, bool backward);
double few_grad_seconds(const Geom& g);
int few_grad_shares(const Geom& g);
size_t few_grad_sums_bytes(const Geom& g);
int few_conv(const Geom& g, bool backward, const float* src, const float* w, float* dst, const Finish& finish, hipStream_t s);
int few_grad(const Geom& g, const float* in, const float* gout, float* partial, float* gw, WgradSum* sum, hipStream_t s);

}  // namespace znn
