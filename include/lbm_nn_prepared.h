/*
 * lbm_nn_prepared.h - C ABI of the network's calls on prepared operands
 * (liblbm.so): convolutions from weights packed once for the kernels, and the
 * network input of a sphere pack formed on the device.  Conventions as in
 * lbm_nn.h.
 */
#ifndef LBM_NN_PREPARED_H
#define LBM_NN_PREPARED_H

#include "lbm_nn.h"

#ifdef __cplusplus
extern "C" {
#endif

/* The forward convolution from packed weights (nn_conv3d_pack_weights), for
 * callers that keep them: bit-identical and faster.  out_kind 0: out is float y;
 * 1, 2: out is bf16 a without and with ReLU, as nn_conv3d_forward_act. */
lbm_status nn_conv3d_packed_bytes(int ci, int co, size_t* bytes);
lbm_status nn_conv3d_forward_packed(const void* x, const void* packed, const float* bias, void* out,
                                    int out_kind, int n, int d, int h, int w_, int ci, int co,
                                    void* stream);

/* Packs w (bf16 [co][27][ci]) for nn_conv3d_forward_packed: flip 0 for the
 * forward convolution (nn_conv3d_packed_bytes(ci, co)); flip 1 for the
 * backward-data convolution, i.e. of the flipped weights, from w itself
 * (nn_conv3d_packed_bytes(co, ci); dx = forward_packed(dy, packed, NULL, ...,
 * ci = co, co = ci)). */
lbm_status nn_conv3d_pack_weights(const void* w, void* packed, int ci, int co, int flip,
                                  void* stream);

/* Network input of a periodic pack of spheres on the grid of half the
 * resolution (the two-grid start): x (bf16, ec,ec,ec,8 with ec = edge / 2) is 1
 * in channel 0 where the coarse node at fine position 2j + 1/2 lies in no sphere
 * or periodic image (strictly inside is solid), 0 elsewhere.  spheres: host
 * double[4 * n], rows cx, cy, cz, r in fine lattice units, read before the call
 * returns; box edge `edge` (even). */
lbm_status nn_coarse_pack_input(const double* spheres, int n, int edge, void* x, void* stream);

#ifdef __cplusplus
}
#endif

#endif
