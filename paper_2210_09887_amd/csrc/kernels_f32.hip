// Launch of the fp32 convolution tile (conv_f32.h).
#include "conv_f32.h"

namespace mdcnn {

__global__ __launch_bounds__(256, 2) void k_conv_f32(TileGrid g, int tiles, unsigned blocks, EdgeBatch eb) {
    // (blockIdx.z: stream of the batch.  The descriptor is not read in one go here: with its fields held in scalar registers the K
    // loop is scheduled worse, ResNet-18-style 256 x 256 frame 630 -> 644 us, 512 x 512 in flight 849 -> 825 frames/s)
    const EdgeDev& e = eb.d[blockIdx.z];
    __shared__ __align__(16) float smem[kF32Smem];
    __shared__ unsigned s_vm[kF32Px], s_or[4];
    __shared__ int sh[8];
    const unsigned nblk = blocks - g.npub - g.ncopy;
    if (blockIdx.x >= nblk) {
        side_block<float>(e, g, blockIdx.x - nblk, reinterpret_cast<unsigned char*>(smem));
        return;
    }
    const bool published = (e.k == 1 || e.k == 3) && !e.up;      // by blocks of their own (the source's list: whenever k is 1 or 3)
    const int nseg = e.up ? 0 : edge_segments(e);         // (an upsampling edge publishes no compute list)
    for (int u = (int)blockIdx.x; u < tiles * g.NT; u += (int)nblk) {
        const int nt = u % g.NT, mt = u / g.NT, ty = mt / g.tiles_x, tx = mt - ty * g.tiles_x;
        __syncthreads();                                  // previous tile is done with LDS
        f32_tile(e, ty * g.p0, tx * g.p1, g.p0, g.p1, nt * kF32Co, published, smem, s_vm, s_or);
        if (nt == 0 && mt < nseg && !published) publish_segment(e, mt, sh);      // (there are at least as many tiles as segments)
    }
    if (e.k != 1 && e.k != 3) carry_source_compaction(e, sh, blockIdx.x, nblk);
}

hipError_t launch_conv_f32(const EdgeBatch& eb, int nb, hipStream_t st, bool* read) {
    const EdgeDev& e = eb.d[0];
    const int ih = e.up ? e.sH : e.Hp, iw = e.up ? e.sW : e.Wp, NT = (e.Cout + kF32Co - 1) / kF32Co;
    int th = 1, tw = 1;
    long long tiles = 0;
    if (!tile_2d(ih, iw, 1, kF32Px, kF32Px, &th, &tw, &tiles)) return hipErrorInvalidValue;     // (never: one pixel always fits)
    const long long items = tiles * NT;
    const unsigned ncopy = e.up ? 0u : copy_blocks(e, 4);
    if (read && ncopy) *read = true;
    const TileGrid g{e.k == 1 || e.k == 3 ? publish_blocks(e) : 0u, ncopy, NT, th, tw, (iw + tw - 1) / tw, 0u, 0u};
    const unsigned blocks = (unsigned)(items < 16384 ? items : 16384) + g.npub + g.ncopy;
    k_conv_f32<<<dim3(blocks, 1, nb), dim3(256), 0, st>>>(g, (int)tiles, blocks, eb);
    return hipGetLastError();
}

// Rows of whole 32-byte blocks, tensors a 32-bit byte offset reaches - but for layers of very few products on a large window,
// which the plain kernel with the weights in LDS (k_conv_ldsw) does sooner: this tile costs its flag, weight and row round
// trips whether a pixel takes 128 products or 8192, and a large window has many tiles.  Where updates come in clusters it
// leaves most tiles at once and the line lies lower than it does for dense frames.  Frames in a row of a one-layer network,
// this kernel / the plain one, in us, all pixels updated and clusters of 24 x 24 pixels on a fifth of the frame:
//   1x1,  8 -> 16, 512 x 512: 120 / 36, 61 / 29;   256 x 256: 38 / 21, 25 / 17;   128 x 128: 19.7 / 16.5, 16.5 / 16.6
//   1x1, 24 -> 32, 512 x 512: 145 / 72, 72 / 60;   224 x 224: 36 / 29, 23 / 22;   128 x 128: 20.2 / 18.6, 16.8 / 16.5
//   1x1, 96 -> 16, 512 x 512: 184 / 110, 88 / 72;  224 x 224: 43 / 31, 26 / 24;   128 x 128 (past the line): 22.9 / 21.6, 18.5 / 19.0
//   3x3,  8 -> 16, 512 x 512: 127 / 51, 56 / 45;   180 x 180: 29 / 22, 20 / 20;   128 x 128 (past): 22.8 / 20.1, 18.0 / 19.0
//   more products (past): 3x3, 8 -> 32, 512 x 512: 132 / 80, 61 / 74; 8 -> 64: 168 / 138, 101 / 132; 24 -> 16, 256 x 256: 48 / 39, 27 / 30
// Into 2 x 2 pixels the plain kernel writes from fewer blocks and needs four times the window (launches alone): 64 -> 16 from 256 x 256
// pixels 36 / 20, 20 / 14; past the line 8 -> 64 from 128 x 128: 16.7 / 17.8, 11.0 / 11.8, 24 -> 32: 15.5 / 14.0, 10.6 / 11.7.
// The choice is made by one video's layer: a video of a batch gives the bits it gives alone.
bool f32_applies(const EdgeDev& e) {
    const long long lim = 1ll << 31, products = (long long)e.k * e.k * e.Cin * e.Cout;
    const long long pixels = e.up ? (long long)e.sH * e.sW : (long long)e.Hp * e.Wp;
    if (products <= 2048 && (e.up ? 64 : 16) * products <= pixels) return false;
    return e.k >= 1 && e.k <= 5 && !e.op && e.Cin % 8 == 0 && (e.Cout % 32 == 0 || e.Cout == 16) &&
           (long long)e.sH * e.sW * e.Cin * 4 < lim && (long long)e.Hp * e.Wp * e.Cout * 4 < lim && products * 4 < lim;
}

}  // namespace mdcnn
