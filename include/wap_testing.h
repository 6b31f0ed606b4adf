/*
 * wap_testing.h -- hooks of libwap that exist for its parity tests only; not part of the product boundary.
 */
#ifndef WAP_TESTING_H
#define WAP_TESTING_H

#ifdef __cplusplus
extern "C" {
#endif

/* Process-wide and NOT thread safe (plain globals read while a plan is made): force the tile configuration of
 * the forward-type kernels (0..9, 8: those of conv_c3.hip; 12 / 14: the patch kernel's flat 64 x 128 / 192 x 64 tiles with
 * the reduction in nsplit >= 2 parts; 15: the few-channel kernel; 100 + a tiling of conv_tile2d_flat.hip; 203: 8 x 28 strips, 204 .. 206: flat 128-channel tiles of 128 .. 192 pixels), of the weight-gradient kernel (0..4; 7: the
 * few-channel kernel; 5 / 6: the patch kernel with two / one
 * 32-channel dy blocks per wavefront) and the number of reduction splits;
 * -1 restores the shape-driven choice.  Forced values that the shape cannot use are ignored, and the
 * *_workspace_bytes queries reflect the forced choice.  Lets the tests reach every kernel and tile
 * configuration with small shapes. */
void wap_debug_force(int fwd_cfg, int wgrad_cfg, int nsplit);

#ifdef __cplusplus
}
#endif
#endif /* WAP_TESTING_H */
