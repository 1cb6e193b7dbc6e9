// Launch of the fp32 convolution tile (conv_f32.h).
#include "conv_f32.h"

namespace mdcnn {

__global__ __launch_bounds__(256, 2) void k_conv_f32(EdgeBatch eb, int NT, int tiles_x, int tiles, int th, int tw) {
    const EdgeDev& e = eb.d[blockIdx.z];                  // blockIdx.z: stream of the batch
    __shared__ __align__(16) float smem[kF32Smem];
    __shared__ unsigned s_vm[kF32Px], s_or[4];
    __shared__ int sh[8];
    const int nseg = e.up ? 0 : edge_segments(e);         // (an upsampling edge publishes no compute list)
    for (int u = blockIdx.x; u < tiles * NT; u += gridDim.x) {
        const int nt = u % NT, mt = u / NT, ty = mt / tiles_x, tx = mt - ty * tiles_x;
        __syncthreads();                                  // previous tile is done with LDS
        f32_tile(e, ty * th, tx * tw, th, tw, nt * kF32Co, smem, s_vm, s_or);
        if (nt == 0 && mt < nseg) publish_segment(e, mt, sh);      // (there are at least as many tiles as segments)
    }
    carry_source_compaction(e, sh);
}

hipError_t launch_conv_f32(const EdgeBatch& eb, int nb, hipStream_t st) {
    const EdgeDev& e = eb.d[0];
    const int ih = e.up ? e.sH : e.Hp, iw = e.up ? e.sW : e.Wp, NT = (e.Cout + kF32Co - 1) / kF32Co;
    int th = 1, tw = 1;
    long long tiles = 0;
    if (!tile_2d(ih, iw, 1, kF32Px, kF32Px, &th, &tw, &tiles)) return hipErrorInvalidValue;     // (never: one pixel always fits)
    const long long items = tiles * NT;
    k_conv_f32<<<dim3((unsigned)(items < 16384 ? items : 16384), 1, nb), dim3(256), 0, st>>>(eb, NT, (iw + tw - 1) / tw, (int)tiles, th, tw);
    return hipGetLastError();
}

// Rows of whole 32-byte blocks, tensors a 32-bit byte offset reaches - but for layers of few products on a large window,
// which the plain kernel with the weights in LDS (k_conv_ldsw) does sooner: this tile costs its flag, weight and row round
// trips whether a pixel takes 128 products or 8192, and a large window has many tiles.  All pixels updated, this kernel /
// the plain one, in us: 1x1, 8 -> 16 channels at 64 x 64: 9.7 / 8.4, 256 x 256: 32.6 / 14.5, 512 x 512: 107 / 23; 72 -> 32 at
// 128 x 128: 14.9 / 13.1, 256 x 256: 34.3 / 22.3; 3x3, 8 -> 64 at 180 x 180: 29.3 / 28.7, 512 x 512: 146 / 115; 1x1, 64 -> 32
// into 2 x 2 pixels at 256 x 256: 36.2 / 26.0.  On the other side of the line: 1x1, 72 -> 64 at 128 x 128: 15.0 / 17.0; 3x3,
// 8 -> 16 at 64 x 64: 12.0 / 13.7; and above 32 KiB of weights the plain kernel has too few blocks: 3x3, 72 -> 16 at 256 x 256:
// 53.9 / 79.6, 40 -> 32: 45.6 / 85.1.  Near the line either may be ahead by a tenth (with few pixels updated the plain one by
// a fifth).  The choice is made by one video's layer: a video of a batch gives the bits it gives alone.
bool f32_applies(const EdgeDev& e) {
    const long long lim = 1ll << 31, products = (long long)e.k * e.k * e.Cin * e.Cout;
    const long long pixels = e.up ? (long long)e.sH * e.sW : (long long)e.Hp * e.Wp;
    if (e.Cout <= 512 && products <= 8192 && 6 * products <= pixels) return false;
    return e.k >= 1 && e.k <= 5 && !e.op && e.Cin % 8 == 0 && (e.Cout % 32 == 0 || e.Cout == 16) &&
           (long long)e.sH * e.sW * e.Cin * 4 < lim && (long long)e.Hp * e.Wp * e.Cout * 4 < lim && products * 4 < lim;
}

}  // namespace mdcnn
