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

// Rows of whole 32-byte blocks, tensors a 32-bit byte offset reaches.
bool f32_applies(const EdgeDev& e) {
    const long long lim = 1ll << 31;
    return e.k >= 1 && e.k <= 5 && !e.op && e.Cin % 8 == 0 && (e.Cout % 32 == 0 || e.Cout == 16) &&
           (long long)e.sH * e.sW * e.Cin * 4 < lim && (long long)e.Hp * e.Wp * e.Cout * 4 < lim && (long long)e.k * e.k * e.Cin * e.Cout * 4 < lim;
}

}  // namespace mdcnn
