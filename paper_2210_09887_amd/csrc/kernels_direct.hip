// Launches of the convolution tile that reads its operands straight from global memory (conv_direct.h).
#include <atomic>

#include "conv_direct.h"

namespace mdcnn {

template <typename T, int TM, int TN>
__global__ __launch_bounds__(256, 2) void k_conv_direct(EdgeBatch eb, int NT, int tiles_x, int tiles) {
    const EdgeDev& e = eb.d[blockIdx.z];                  // blockIdx.z: stream of the batch
    using Cfg = DirectCfg<T, TM, TN>;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ unsigned s_vm[Cfg::PX];
    __shared__ int sh[8];
    const int nseg = e.up ? 0 : edge_segments(e);         // (an upsampling edge publishes no compute list)
    for (int u = blockIdx.x; u < tiles * NT; u += gridDim.x) {
        const int nt = u % NT, mt = u / NT, ty = mt / tiles_x, tx = mt - ty * tiles_x;
        __syncthreads();                                  // previous tile is done with LDS
        direct_tile<T, TM, TN>(e, ty * Cfg::TH, tx * Cfg::TW, nt * Cfg::CO, reinterpret_cast<float*>(smem), s_vm);
        if (nt == 0 && mt < nseg) publish_segment(e, mt, sh);      // (there are at least as many tiles as segments)
    }
    carry_source_compaction(e, sh);
}

template <typename T, int TM, int TN>
static hipError_t launch_direct_t(const EdgeBatch& eb, int nb, hipStream_t st) {
    const EdgeDev& e = eb.d[0];
    using Cfg = DirectCfg<T, TM, TN>;
    auto kern = k_conv_direct<T, TM, TN>;
    static std::atomic<bool> attr_set{false};
    if (Cfg::SMEM > 49152 && !attr_set.load(std::memory_order_acquire)) {
        const hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, Cfg::SMEM);
        if (err != hipSuccess) { (void)hipGetLastError(); return err; }    // do not leave it for the next call to report
        attr_set.store(true, std::memory_order_release);
    }
    const int ih = e.up ? e.sH : e.Hp, iw = e.up ? e.sW : e.Wp;
    const int tx = (iw + Cfg::TW - 1) / Cfg::TW, ty = (ih + Cfg::TH - 1) / Cfg::TH, NT = (e.Cout + Cfg::CO - 1) / Cfg::CO;
    const long long items = (long long)tx * ty * NT;
    kern<<<dim3((unsigned)(items < 16384 ? items : 16384), 1, nb), dim3(256), Cfg::SMEM, st>>>(eb, NT, tx, tx * ty);
    return hipGetLastError();
}

template <typename T>
static hipError_t launch_direct_n(const EdgeBatch& eb, int nb, hipStream_t st) {
    const EdgeDev& e = eb.d[0];
    const long long px = e.up ? (long long)e.sH * e.sW : (long long)e.Hp * e.Wp;
    // the largest tile that still gives every compute unit two (a tile's sums do not depend on its size)
    auto tiles = [&](int p, int c) { return ((px + p - 1) / p) * ((e.Cout + c - 1) / c) * nb; };
    if (e.Cout % 64 == 0 && tiles(64, 64) >= 512) return launch_direct_t<T, 2, 2>(eb, nb, st);
    if (e.Cout % 64 == 0 && tiles(32, 64) >= 512) return launch_direct_t<T, 1, 2>(eb, nb, st);
    return launch_direct_t<T, 1, 1>(eb, nb, st);
}

// Rows of whole 32-byte K blocks, tensors a 32-bit byte offset reaches.
bool direct_applies(const EdgeDev& e, int dtype) {
    const long long es = dtype == MDCNN_F16 ? 2 : 4, lim = 1ll << 31;
    return e.k >= 1 && e.k <= 5 && !e.op && (e.Cin * es) % 32 == 0 && (e.Cout % 32 == 0 || e.Cout == 16) &&
           (long long)e.sH * e.sW * e.Cin * es < lim && (long long)e.Hp * e.Wp * e.Cout * es < lim && (long long)e.k * e.k * e.Cin * e.Cout * es < lim;
}

hipError_t launch_conv_direct(const EdgeBatch& eb, int nb, int dtype, hipStream_t st) {
    return dtype == MDCNN_F16 ? launch_direct_n<f16>(eb, nb, st) : launch_direct_n<float>(eb, nb, st);
}

}  // namespace mdcnn
