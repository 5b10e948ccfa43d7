// FFT method on overlapping tiles (fft_tile.hip): the tiling of a layer and the three passes on it.
#pragma once

#include "znn_internal.h"

namespace znn {

// the library's choice of tile lengths for a layer whose kernel spectra may take `spectra_bytes` (on = false: none does)
Tiling tile_search(const Geom& g, size_t spectra_bytes);
size_t tile_kernel_bytes(const Geom& g, const Tiling& L);               // spectra of all kernels
size_t tile_node_bytes(const Geom& g, const Tiling& L, int maps);       // spectra of `maps` images or gradients
size_t tile_workspace_bytes(const Geom& g, const Tiling& L, int pass, bool resident);
int tile_kernel_spectra(const Geom& g, const Tiling& L, const float* w, float2* What, hipStream_t s);
// ws: tile_workspace_bytes of the pass; forward: ws_bytes, at least the kernels' spectra (where they are to lie there) and those of one tile; finish: the rectifier only
int tile_fwd(const Geom& g, const Tiling& L, const float* in, const KernelSpectra& kernels, float* out,
             void* ws, size_t ws_bytes, float2* memo_in, const Finish& finish, hipStream_t s);
// The kernel gradient beside the backward pass, from the kept spectra U of the images and those of the gradients that the pass makes (memo_gout), where gw
// is not NULL; tile_joined_bytes: the workspace then, 0: not of this layer.
struct TileGrad { const float2* U; float* gw; };
size_t tile_joined_bytes(const Geom& g, const Tiling& L);
int tile_bwd(const Geom& g, const Tiling& L, const float* gout, const KernelSpectra& kernels, float* gin,
             void* ws, float2* memo_gout, const Finish& finish, const TileGrad& grad, hipStream_t s);
int tile_wgrad(const Geom& g, const Tiling& L, const float* in, const float* gout, float* gw, void* ws, hipStream_t s);
int tile_wgrad_from_spectra(const Geom& g, const Tiling& L, const float2* U, const float2* V, float* gw, void* scratch,
                            hipStream_t s);

}  // namespace znn
