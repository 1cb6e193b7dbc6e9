// Launch of the fp32 convolution tile (conv_f32.h).
#include <atomic>

#include "conv_f32s.h"

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

template <typename Cfg>
__global__ __launch_bounds__(256, Cfg::MINB) void k_conv_f32s(TileGrid g, unsigned blocks, EdgeBatch eb) {
    extern __shared__ __align__(16) unsigned char smem[];
    const unsigned nblk = blocks - g.npub - g.ncopy;
    if (blockIdx.x >= nblk) side_block<float>(eb.d[blockIdx.z], g, blockIdx.x - nblk, smem);
    else split_tile<Cfg>(eb.d[blockIdx.z], blockIdx.x, g);
}

template <typename Cfg>
static hipError_t launch_split(const EdgeBatch& eb, int nb, hipStream_t st, bool* done, bool* read) {
    const EdgeDev& e = eb.d[0];
    int th, tw;
    long long tiles;
    rect_tile(e.Hp, e.Wp, Cfg::M, Cfg::ROWS, 1, &th, &tw, &tiles);
    const int NT = e.Cout / 32, tiles_x = (e.Wp + tw - 1) / tw;
    *done = (double)tiles * NT * NT < 4e9 && (double)tiles * tiles_x < 4e9;      // (the reciprocals are exact below 2^32)
    if (!*done) return hipSuccess;
    const unsigned npub = publish_blocks(e), ncopy = copy_blocks(e, 4), blocks = (unsigned)(tiles * NT) + npub + ncopy;
    if (read && ncopy) *read = true;
    const TileGrid g{npub, ncopy, NT, th, tw, tiles_x, reciprocal_of((unsigned)NT), reciprocal_of((unsigned)tiles_x)};
    auto kern = k_conv_f32s<Cfg>;
    static std::atomic<bool> attr_set{false};
    if (!attr_set.load(std::memory_order_acquire)) {
        hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, Cfg::SMEM);
        if (err != hipSuccess) { (void)hipGetLastError(); return err; }    // do not leave it for the next call to report
        attr_set.store(true, std::memory_order_release);
    }
    kern<<<dim3(blocks, 1, nb), dim3(256), Cfg::SMEM, st>>>(g, blocks, eb);
    return hipGetLastError();
}

// Row tiles of a tile: what the compute unit with the most tiles takes, a tile's start and end and its steps one behind the other (a
// compute unit issues the steps of two tiles in the time of both).  Measured as in conv_f32s.h, us a frame with 1 / 2 / 3: 64 -> 32 on
// 16 x 16 10.0 / 11.3 / 12.4, 192 -> 96 on 37 x 53 18.3 / 21.0 / 25.2, 512 -> 512 on 8 x 8 27.8 / 35.6 / 37.6; 64 -> 64 on 64 x 64
// 13.4 / 13.1 / 15.2, on 128 x 128 28.7 / 25.4 / 29.7, on 256 x 256 82.5 / 65.9 / 82.3, 256 -> 256 on 32 x 32 26.5 / 24.7 / 29.5;
// 128 -> 128 on 64 x 64 23.6 / 23.4 / 22.8, 512 -> 512 on 32 x 32 82.2 / 62.2 / 58.0.
int split_choice(int Hp, int Wp, int Cin, int Cout, int nb) {
    constexpr double start[3] = {2.6, 3.5, 5.0}, step[3] = {0.22, 0.34, 0.62};
    int best = 0;
    double least = 0;
    for (int tm = 1; tm <= 3; ++tm) {
        int th, tw;
        long long tiles;
        rect_tile(Hp, Wp, 32 * tm, split_rows(tm), 1, &th, &tw, &tiles);
        const double per_cu = (double)tiles * (Cout / 32) * nb / 256;
        const double cost = (per_cu > 4 ? per_cu : (double)(int)(per_cu + 0.9999)) * (start[tm - 1] + 9.0 * (Cin / 64) * step[tm - 1]);
        if (!best || cost < least) { best = tm; least = cost; }
    }
    return best;
}

hipError_t launch_conv_f32(const EdgeBatch& eb, int nb, hipStream_t st, bool* read) {
    const EdgeDev& e = eb.d[0];
    if (e.k == 3 && e.stride == 1 && e.Cin % 64 == 0 && e.Cout % 32 == 0) {
        bool done = false;
        hipError_t err;
        switch (split_choice(e.Hp, e.Wp, e.Cin, e.Cout, nb)) {
            case 1: err = launch_split<SplitCfg<1>>(eb, nb, st, &done, read); break;
            case 2: err = launch_split<SplitCfg<2>>(eb, nb, st, &done, read); break;
            default: err = launch_split<SplitCfg<3>>(eb, nb, st, &done, read); break;
        }
        if (done) return err;
    }
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
