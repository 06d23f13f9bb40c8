// Layer kernels the network object uses beside those of include/unet.h: backward steps
// with the ReLU mask of the tensor they write applied on the way out (m, rows of ldm, from
// channel offm: the activation whose gradient is written; entries where it is not
// positive become zero), and the transposed weights of several layers in one launch.
// Arguments and status codes as in include/unet.h.
#pragma once

#include <cstdint>

namespace unet {

// dx = conv(dy, wt) without bias, masked
int conv3d_dgrad_relu(const uint16_t *dy, int ldy, int offy, const uint16_t *wt, uint16_t *dx, int ldx, int offx,
                      const uint16_t *m, int ldm, int offm, int nz, int ny, int nx, int cout, int cin, void *stream);
// unet_up_bwd and unet_pool_bwd, masked
int up_bwd_relu(const uint16_t *dy, int ldy, int offy, uint16_t *dx, int ldx, int offx, const uint16_t *m, int ldm,
                int offm, int nz, int ny, int nx, int c, void *stream);
int pool_bwd_relu(const uint16_t *dy, int ldy, int offy, uint16_t *dx, int ldx, int offx, const uint16_t *m, int ldm,
                  int offm, int nz, int ny, int nx, int c, void *stream);
// unet_head_bwd with dx masked by the head's own input x
int head_bwd_relu(const uint16_t *x, int ldx, const float *w, const float *dout, uint16_t *dx, float *dw, float *db,
                  int64_t nvox, int c, void *stream);

// unet_conv3d_wtrans of n layers (w + w_off[l] -> wt + wt_off[l])
constexpr int kMaxTrans = 16;
struct TransTable {
    int n;
    int cin[kMaxTrans], cout[kMaxTrans];
    int64_t w_off[kMaxTrans], wt_off[kMaxTrans];
};
int conv3d_wtrans_all(const uint16_t *w, uint16_t *wt, const TransTable &t, void *stream);

}  // namespace unet
