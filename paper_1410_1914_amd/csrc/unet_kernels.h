// Layer kernels the network object uses beside those of include/unet.h: backward steps
// with the ReLU mask of the tensor they write applied on the way out (m, rows of ldm, from
// channel offm: the activation whose gradient is written; entries where it is not
// positive become zero), and convolutions with their weights laid out for the kernels.
// Arguments and status codes as in include/unet.h.
#pragma once

#include <cstdint>

namespace unet {

// A 3x3x3 convolution (unet_conv3d_fwd, or unet_conv3d_fwd_cat where x2 is not null) with
// weights in fragment order and the ReLU mask m on what is written (unless null)
struct Conv {
    const uint16_t *x;
    int ldx;
    const uint16_t *w;
    const float *b;
    uint16_t *y;
    int ldy, relu;
    const uint16_t *x2 = nullptr;
    int ldx2 = 0, cin1 = 0;
    const uint16_t *m = nullptr;
    int ldm = 0, offm = 0;
};
int conv3d(const Conv &c, int nz, int ny, int nx, int cin, int cout, void *stream);
// unet_up_bwd and unet_pool_bwd, masked
int up_bwd_relu(const uint16_t *dy, int ldy, int offy, uint16_t *dx, int ldx, int offx, const uint16_t *m, int ldm,
                int offm, int nz, int ny, int nx, int c, void *stream);
int pool_bwd_relu(const uint16_t *dy, int ldy, int offy, uint16_t *dx, int ldx, int offx, const uint16_t *m, int ldm,
                  int offm, int nz, int ny, int nx, int c, void *stream);
// unet_head_bwd with dx masked by the head's own input x
int head_bwd_relu(const uint16_t *x, int ldx, const float *w, const float *dout, uint16_t *dx, float *dw, float *db,
                  int64_t nvox, int c, void *stream);

// Weights in fragment order for layers of cin -> cout channels: w + from holds rows of
// unet_kpad(cin) as unet_conv3d_fwd reads them or, transposed, the cin rows of
// unet_kpad(cout) of the layer whose backward data convolution this is.
constexpr int kMaxPack = 27;
struct PackLayer {
    int cin, cout, transposed;
    int64_t from, to;
};
struct PackTable {
    int n;
    PackLayer l[kMaxPack];
};
int64_t conv3d_packed_len(int cin, int cout);
int conv3d_pack(const uint16_t *w, uint16_t *packed, const PackTable &t, void *stream);

}  // namespace unet
