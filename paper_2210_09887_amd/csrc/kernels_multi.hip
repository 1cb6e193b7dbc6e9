// Convolutions of several independent edges in one launch: the branches of a multi-resolution network between two fusion
// points.  Each is a launch of 12 to 110 blocks that takes the latency of one tile (about 12 us, whatever its size), so one
// after the other they leave the chip idle and cost the host a launch each; on streams of their own every crossing costs
// an event.  A block finds its edge by its number and runs the tile its edge would run alone: the results are the same bits.
#include <atomic>

#include "conv_rect.h"
#include "conv_tiles.h"
#include "conv_up.h"

namespace mdcnn {

__global__ __launch_bounds__(256, 2) void k_conv_multi(unsigned b1, unsigned b2, unsigned b3, unsigned b4, unsigned b5, unsigned videos, ConvMulti m) {
    unsigned blk;
    const int j = find_job(b1, b2, b3, b4, b5, blockIdx.x, &blk);
    const ConvJob& jb = m.job[j];
    ConvVid v = m.vid[j * (int)videos + (int)blockIdx.z];
    EdgeDev e = jb.e;
    TileGrid g = jb.g;
    unsigned blocks = jb.blocks;
    int body = jb.body, items = jb.items;
    read_now(v.sd, v.dd, v.p_oy, v.p_ox, blocks, body, items, g.npub, g.NT, g.p0, g.p1, g.tiles_x, g.per_NT, g.per_tiles_x, e.delta, e.sflags, e.sH, e.sW,
             e.Cin, e.P, e.Cout, e.Hp, e.Wp, e.by0, e.bx0, e.w, e.wp, e.k, e.stride, e.pad, e.up);
    if (blk >= blocks) return;                            // (the numbers between two edges, up to a multiple of 8)
    auto at = [](auto*& p, long long d) {
        if (p) p = (std::remove_reference_t<decltype(p)>)((uintptr_t)p + (uintptr_t)d);
    };
    at(e.delta, v.sd); at(e.sflags, v.sd); at(e.pub_list, v.sd); at(e.pub_lcnt, v.sd); at(e.pub_lacc, v.sd); at(e.scounters, v.sd);
    at(e.P, v.dd); at(e.dflags, v.dd); at(e.clist, v.dd); at(e.ccnt, v.dd); at(e.cacc, v.dd); at(e.dcounters, v.dd);
    e.p_oy = v.p_oy;
    e.p_ox = v.p_ox;
    const unsigned nblk = blocks - g.npub;
    if (blk >= nblk) {                                    // (once for all bodies: the code of a launch is fetched anew)
        publish_edge(e, blk - nblk, g.npub);
        return;
    }
#define RECT(M, TN)                                                                                                       \
    case multi_rect_body(M, TN): rect_body<RectTiles<TN>::T##M, false>(e, blk, g); break;
#define RECT_S2(T, TN)                                                                                                    \
    case multi_rect_body(kRect##T, TN): rect_body<RectTiles<TN>::T, false>(e, blk, g); break;
#define HALO(NSUB, WMV, WK, TM, TN, KC, NLD, RING, T2D)                                                                   \
    case multi_halo_body(NSUB, WMV, WK, TM, TN, KC, NLD, RING, T2D):                                                      \
        halo_body<NSUB, WMV, WK, TM, TN, KC, NLD, 3, RING, 2, T2D>(e, blk, nblk, g.NT, items, g.p0, g.p1);               \
        break;
#define TILED(WM, WN, TM, TN, KC)                                                                                         \
    case multi_tiled_body(WM, WN, TM, TN, KC, 1): tiled_body<WM, WN, TM, TN, KC, 1, false>(e, blk, nblk, g, items); break;
    switch (body) {
        RECT(64, 1) RECT(64, 2) RECT(96, 1) RECT(96, 2) RECT(128, 1) RECT(128, 2)
        RECT_S2(S2One, 1) RECT_S2(S2One, 2) RECT_S2(S2One, 4) RECT_S2(S2, 1) RECT_S2(S2, 2) RECT_S2(S2, 4) RECT_S2(S2Half, 1) RECT_S2(S2Half, 2)
        HALO(2, 2, 2, 2, 1, 32, 3, 3, true)
        HALO(4, 2, 2, 1, 1, 32, 2, 9, true)
        TILED(2, 2, 1, 1, 32) TILED(2, 2, 1, 1, 64) TILED(2, 2, 1, 1, 128)
        TILED(4, 1, 1, 1, 32) TILED(4, 1, 1, 1, 64) TILED(4, 1, 1, 1, 128)
        TILED(2, 2, 2, 1, 32) TILED(2, 2, 2, 1, 64) TILED(2, 2, 2, 1, 128)
        TILED(2, 2, 1, 2, 32) TILED(2, 2, 1, 2, 64) TILED(2, 2, 1, 2, 128)
        TILED(2, 2, 2, 2, 32) TILED(2, 2, 2, 2, 64) TILED(2, 2, 2, 2, 128)
        case kMultiUpBody: up_body<false>(e, blk, g); break;
        default: break;
    }
#undef RECT
#undef RECT_S2
#undef HALO
#undef TILED
}

hipError_t launch_conv_multi(ConvMulti& m, int videos, unsigned smem, hipStream_t st) {
    m.blocks.clear();
    m.videos = videos;
    for (int j = 0; j < m.n; ++j) m.blocks.add(j, (m.job[j].blocks + 7u) & ~7u);
    static std::atomic<bool> attr_set{false};
    if (smem > 32768 && !attr_set.load(std::memory_order_acquire)) {
        const hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void*>(k_conv_multi), hipFuncAttributeMaxDynamicSharedMemorySize, 80 * 1024);
        if (err != hipSuccess) { (void)hipGetLastError(); return err; }    // do not leave it for the next call to report
        attr_set.store(true, std::memory_order_release);
    }
    if (smem > 80u * 1024u) return hipErrorInvalidValue;
    k_conv_multi<<<dim3(m.blocks.total, 1, (unsigned)videos), dim3(256), smem, st>>>(m.blocks.begin[1], m.blocks.begin[2], m.blocks.begin[3], m.blocks.begin[4], m.blocks.begin[5],
                                                                                                (unsigned)videos, m);
    return hipGetLastError();
}

}  // namespace mdcnn
