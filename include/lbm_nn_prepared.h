/*
 * lbm_nn_prepared.h - C ABI of the network's calls on prepared operands
 * (liblbm.so): convolutions from weights packed once for the kernels, steps of
 * the network fused with their neighbours, and the network input of a sphere
 * pack formed on the device.  Conventions as in lbm_nn.h.
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

/* nn_conv3d_pack_weights of `count` layers in few launches. */
typedef struct {
  const void* w;
  void* packed;
  int ci, co, flip;
} nn_pack_item;
lbm_status nn_conv3d_pack_weights_many(const nn_pack_item* items, int count, void* stream);

/* nn_adam of `count` tensors in few launches (w_bf16 may be NULL); both lists
 * are read before the call returns, and no tensor may be listed twice. */
typedef struct {
  float* w;
  const float* g;
  float* m1;
  float* m2;
  void* w_bf16;
  long long n;
} nn_adam_tensor;
lbm_status nn_adam_many(const nn_adam_tensor* tensors, int count, float lr, float b1, float b2,
                        float eps, int step, void* stream);

/* Network input of a periodic pack of spheres on the grid of half the
 * resolution (the two-grid start): x (bf16, ec,ec,ec,8 with ec = edge / 2) is 1
 * in channel 0 where the coarse node at fine position 2j + 1/2 lies in no sphere
 * or periodic image (strictly inside is solid), 0 elsewhere.  spheres: host
 * double[4 * n], rows cx, cy, cz, r in fine lattice units, read before the call
 * returns; box edge `edge` (even). */
lbm_status nn_coarse_pack_input(const double* spheres, int n, int edge, void* x, void* stream);

/* y = [u | b] along channels (bf16, n,2d,2h,2w,ca+cb), u the upsampled coarse a
 * (bf16, n,d,h,w,ca) and b (bf16, n,2d,2h,2w,cb): nn_upsample2_forward and
 * nn_concat_channels without the upsampled tensor.  ca and cb multiples of 8,
 * 16-byte aligned pointers, fewer than 2^31 output elements. */
lbm_status nn_upsample_concat(const void* a, const void* b, void* y, int n, int d, int h, int w_,
                              int ca, int cb, void* stream);

/* The gradient of a of nn_upsample_concat (float da n,d,h,w,ca) from that of y
 * (float dcat n,2d,2h,2w,ca+cb): nn_split_channels' first part through
 * nn_upsample2_backward.  ca and cb multiples of 4, limits as above. */
lbm_status nn_concat_upsample_backward(const float* dcat, float* da, int n, int d, int h, int w_,
                                       int ca, int cb, void* stream);

/* nn_relu_backward_bias for a layer whose output (n,d,h,w,c) feeds a pooling and
 * the skip part of a concatenation: its gradient is nn_pool2_backward(pooled) +
 * the last c channels of cat, pooled float (n,d/2,h/2,w/2,c) and cat float
 * (n,d,h,w,ca+c) the gradients of the pooled and the concatenated tensor; it is
 * never stored.  Bit-identical to nn_pool2_backward, nn_split_channels, nn_add
 * and nn_relu_backward_bias.  Even d, h, w; c a multiple of 4 up to 1024, ca of
 * 4; n d h w max(d, h, w) up to 2^32, fewer than 2^31 elements in cat, 16-byte
 * aligned pointers (a and dz 8). */
lbm_status nn_pooled_backward_bias(const float* pooled, const float* cat, int ca, const void* a,
                                   void* dz, float* db, void* ws, size_t ws_bytes, int n, int d,
                                   int h, int w_, int c, int relu, void* stream);

#ifdef __cplusplus
}
#endif

#endif
