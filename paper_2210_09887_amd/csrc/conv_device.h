// Device helpers shared by the convolution kernels: list entries, tap masks, the
// per-tile prologue, buffer loads.
#pragma once

#include "mdcnn_internal.h"

namespace mdcnn {

typedef _Float16 f16;
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ int wrapc(int v, int n) { return v >= n ? v - n : v; }

// Division by a number known on the host.
inline unsigned reciprocal_of(unsigned d) { return d > 1 ? 0xffffffffu / d + 1 : 0u; }
__device__ __forceinline__ int by_reciprocal(int a, unsigned r) { return r ? (int)__umulhi((unsigned)a, r) : a; }     // a * divisor < 2^32

// Buffer loads: the address is a resource (base, size) in scalar registers + a per-lane byte offset + a
// scalar byte offset, so a wave spends one vector register on all the addresses of a tensor instead of a
// 64-bit pointer per load (reads past `bytes` return zero instead of faulting).
using rsrc_t = __amdgpu_buffer_rsrc_t;
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ rsrc_t make_rsrc(const void* p, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ f16x8 buf_load16(rsrc_t r, unsigned lane_bytes, unsigned wave_bytes) {
    const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)lane_bytes, (int)wave_bytes, 0);
    return __builtin_bit_cast(f16x8, v);
}

__device__ __forceinline__ size_t pdst_offset(const EdgeDev& e, int wy, int wx) {
    int py = wrapc(e.p_oy + wy, e.Hp), px = wrapc(e.p_ox + wx, e.Wp);
    return ((size_t)py * e.Wp + px) * e.Cout;
}

// Decode list entry -> conv-output coordinates (cy, cx) in the source-aligned
// frame and the top-left destination window pixel (wy, wx).
__device__ __forceinline__ void decode_entry(const EdgeDev& e, int idx, int& cy, int& cx, int& wy, int& wx) {
    if (e.up) {                       // entry = updated source pixel (1x1 conv)
        cy = div24(idx, e.sW, rcp_of(e.sW)); cx = idx - cy * e.sW;
        wy = (cy << e.up) + e.by0; wx = (cx << e.up) + e.bx0;
    } else {                          // entry = destination padded-window pixel (borders may take a window past 2^24 pixels)
        wy = (long long)e.Hp * e.Wp < 1 << 24 ? div24(idx, e.Wp, rcp_of(e.Wp)) : idx / e.Wp;
        wx = idx - wy * e.Wp;
        cy = wy - e.by0; cx = wx - e.bx0;
    }
}

// Update flags of the K x K footprint of output (cy, cx) as a bit mask.  All loads go out together
// (a pixel outside the source reads flag 0 of the site and is masked afterwards).
template <int K>
__device__ __forceinline__ unsigned tap_mask_k(const EdgeDev& e, int cy, int cx) {
    const int y0 = cy * e.stride - e.pad, x0 = cx * e.stride - e.pad;
    unsigned f[K * K];
#pragma unroll
    for (int t = 0; t < K * K; ++t) {
        const int iy = y0 + t / K, ix = x0 + t % K;
        const bool ok = iy >= 0 && iy < e.sH && ix >= 0 && ix < e.sW;
        const unsigned v = e.sflags[ok ? iy * e.sW + ix : 0];
        f[t] = ok ? v : 0u;
    }
    unsigned m = 0;
#pragma unroll
    for (int t = 0; t < K * K; ++t) m |= ((f[t] >> 2) & 1u) << t;      // kFlagM == 4
    return m;
}

// The same for three by three, a row of three flags at a time: one word, which need not be aligned and may start or end beyond
// the flags of the site (the regions before and behind them in its memory; those bits are masked).  Rows outside the source
// are read from beyond the end of everything, which gives zeros.
struct Taps3 {
    unsigned w[3], cols;              // flag M of the columns inside the source, a byte each
};
__device__ __forceinline__ rsrc_t taps3_rsrc(const uint8_t* sflags, int HW) { return make_rsrc(sflags - 4, (unsigned)HW + 7u); }
__device__ __forceinline__ void taps3_load(rsrc_t rs, int sH, int sW, int iy, int ix, bool in, Taps3& t) {    // (iy, ix): the top left tap
    t.cols = 0;
#pragma unroll
    for (int c = 0; c < 3; ++c) t.cols |= in && (unsigned)(ix + c) < (unsigned)sW ? (unsigned)kFlagM << (8 * c) : 0u;
#pragma unroll
    for (int r = 0; r < 3; ++r)
        t.w[r] = __builtin_amdgcn_raw_buffer_load_b32(rs, (unsigned)(iy + r) < (unsigned)sH && t.cols ? (iy + r) * sW + ix + 4 : (int)0x80000000u, 0, 0);
}
__device__ __forceinline__ unsigned tap_mask3(const EdgeDev& e, int cy, int cx) {
    Taps3 t;
    taps3_load(taps3_rsrc(e.sflags, e.sH * e.sW), e.sH, e.sW, cy * e.stride - e.pad, cx * e.stride - e.pad, true, t);
    unsigned m = 0;
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        const unsigned b = (t.w[r] & t.cols) >> 2;         // kFlagM == 4
        m |= ((b | b >> 7 | b >> 14) & 7u) << (3 * r);
    }
    return m;
}

__device__ __forceinline__ unsigned tap_mask(const EdgeDev& e, int cy, int cx) {
    switch (e.k) {
        case 1: return tap_mask_k<1>(e, cy, cx);
        case 3: return tap_mask3(e, cy, cx);
        case 5: return tap_mask_k<5>(e, cy, cx);
        default: break;
    }
    unsigned m = 0;
    const int y0 = cy * e.stride - e.pad, x0 = cx * e.stride - e.pad;
    for (int jy = 0; jy < e.k; ++jy) {
        const int iy = y0 + jy;
        const bool yok = iy >= 0 && iy < e.sH;
        for (int jx = 0; jx < e.k; ++jx) {
            const int ix = x0 + jx;
            const bool ok = yok && ix >= 0 && ix < e.sW;
            const unsigned f = ok ? e.sflags[iy * e.sW + ix] : 0u;
            m |= ((f >> 2) & 1u) << (jy * e.k + jx);
        }
    }
    return m;
}

// Number of list segments an edge walks: upsampling edges walk the source
// pixels (view order), all others the destination's padded window.
__device__ __forceinline__ int edge_segments(const EdgeDev& e) {
    const int n = e.up ? e.sH * e.sW : e.Hp * e.Wp;
    return (n + kSegPixels - 1) / kSegPixels;
}

// Statistics: add taps x Cin x Cout to one of the partial multiply-accumulate
// sums of the destination (which: 0 MFMA kernels, 1 plain kernels).
__device__ __forceinline__ void add_macs(const EdgeDev& e, long long taps, int which) {
    if (taps)
        atomicAdd(reinterpret_cast<unsigned long long*>(e.dcounters) + kAccMacsSpread + 8 * which + (blockIdx.x & 7),
                  (unsigned long long)taps * (unsigned long long)(e.Cin * e.Cout));
}
// Sum over the wave, in every lane: moves within the vector unit (row_shr 1, 2, 4, 8, then row_bcast 15 and 31), where a
// shuffle goes through LDS (0.1 us each, six of them in a row: with step 1's, ResNet-18-style 512 x 512 frame 387 -> 380 us,
// 256 x 256 in fp32 666 -> 659, bottleneck 47.3 -> 46.2).
__device__ __forceinline__ int wave_sum(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
    return __builtin_amdgcn_readlane(v, 63);
}

__device__ __forceinline__ unsigned wave_or(unsigned v) {
    v |= __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);
    v |= __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v |= __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v |= __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v |= __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
    v |= __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
    return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}

// Marks a window pixel as touched, if it is in the view: an atomic OR on the word that holds the flag byte, its result
// unused: nothing comes back to the wave, so the loads that follow do not queue behind a read-modify-write round trip
// (the flag region is 256-byte aligned).
__device__ __forceinline__ void mark_pixel(const EdgeDev& e, int wy, int wx) {
    if (!e.dflags) return;
    const int oy = wy - e.by0, ox = wx - e.bx0;
    if (oy >= 0 && oy < e.dH && ox >= 0 && ox < e.dW) {
        const int idx = oy * e.dW + ox;
        atomicOr(reinterpret_cast<unsigned*>(e.dflags + (idx & ~3)), (unsigned)kFlagU << (8 * (idx & 3)));
    }
}
__device__ __forceinline__ void mark_touched(const EdgeDev& e, int wy, int wx) {
    const int f = 1 << e.up;
    for (int a = 0; a < f; ++a)
        for (int b = 0; b < f; ++b) mark_pixel(e, wy + a, wx + b);
}

// Per-tile prologue shared by all convolution kernels.  Thread t looks at index
// seg * kSegPixels + t of the edge's index space, gathers the update flags of its
// footprint (they become the tap mask), and the block ranks the non-empty ones
// with ballot + popcount: the rank is the position in the segment's compute list.
// Entries with rank in [first, first + bm) are decoded into the LDS rows
// s_base / s_wy / s_wx / s_vm (s_vm = 0 beyond the live rows).  With `publish`
// the segment is also written to the destination's compute list.  `touch` marks
// the destination pixels as touched.  Returns the number of entries of the
// segment; sh[4] = valid taps of the tile, sh[5] = OR of its tap masks.
// Block-uniform; two barriers; the caller must have a barrier before the call.
__device__ __forceinline__ int tile_prologue(const EdgeDev& e, int seg, int first, int bm, bool publish, bool touch,
                                             int* s_base, int* s_wy, int* s_wx, unsigned* s_vm, int* sh) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = e.up ? e.sH * e.sW : e.Hp * e.Wp;
    const int p = seg * kSegPixels + tid;
    if (tid < bm) s_vm[tid] = 0;
    if (tid == 0) { sh[4] = 0; sh[5] = 0; }
    int cy = 0, cx = 0, wy = 0, wx = 0;
    unsigned vm = 0;
    if (p < n) {
        decode_entry(e, p, cy, cx, wy, wx);
        if (e.k == 0) vm = (cy >= 0 && cy < e.sH && cx >= 0 && cx < e.sW && (e.sflags[cy * e.sW + cx] & kFlagM)) ? 1u : 0u;
        else if (e.op && (cy < 0 || cy >= e.dH || cx < 0 || cx >= e.dW)) vm = 0;     // pooling outputs exist inside the view only
        else vm = tap_mask(e, cy, cx);
    }
    const bool has = vm != 0;
    const unsigned long long bal = __ballot(has);
    const int rank = __popcll(bal & ((1ull << lane) - 1ull));
    if (lane == 0) sh[wave] = __popcll(bal);
    __syncthreads();
    int off = rank;
    for (int i = 0; i < wave; ++i) off += sh[i];
    const int tot = sh[0] + sh[1] + sh[2] + sh[3];
    const int r = off - first;
    const bool mine = has && r >= 0 && r < bm;
    if (mine) {
        s_vm[r] = vm;
        s_base[r] = (cy * e.stride - e.pad) * e.sW + (cx * e.stride - e.pad);
        s_wy[r] = wy;
        s_wx[r] = wx;
        if (touch) mark_touched(e, wy, wx);
    }
    if (publish && has) e.clist[seg * kSegPixels + off] = p;
    if (publish && tid == 0) {                             // single writer per segment: no atomics
        e.ccnt[seg] = tot;
        e.cacc[seg] += (unsigned long long)tot;
    }
    const unsigned orm = wave_or(mine ? vm : 0u);
    const int taps = wave_sum(mine ? __popc(vm) : 0);
    if (lane == 0 && orm) { atomicOr(reinterpret_cast<unsigned*>(&sh[5]), orm); atomicAdd(&sh[4], taps); }
    __syncthreads();
    return tot;
}

// The first edge of a forward call also compacts the update mask of the source
// site into its list L (segment-local, ascending) and adds up the per-frame
// statistics.  Called by all threads of every block before their own work.
// (blk, nblk: this block's number among those of the edge)
__device__ __forceinline__ void carry_source_compaction(const EdgeDev& e, int* sh, unsigned blk = blockIdx.x, unsigned nblk = gridDim.x) {
    if (!e.pub_list || blockIdx.y != 0) return;
    const int HW = e.sH * e.sW;
    const int nseg = (HW + kSegPixels - 1) / kSegPixels;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int seg = (int)blk; seg < nseg; seg += (int)nblk) {
        const int p = seg * kSegPixels + tid;
        const int f = p < HW && tid < kSegPixels ? e.sflags[p] : 0;       // waves beyond the fourth only keep the barriers
        const unsigned long long bm = __ballot(f & kFlagM), bc = __ballot(f & kFlagC);
        __syncthreads();                                   // sh is free again
        if (lane == 0 && wave < 4) { sh[wave] = __popcll(bm); sh[4 + wave] = __popcll(bc); }
        __syncthreads();
        int off = __popcll(bm & ((1ull << lane) - 1ull));
        for (int i = 0; i < wave; ++i) off += sh[i];
        if (f & kFlagM) e.pub_list[seg * kSegPixels + off] = p;
        if (tid == 0) {                                    // single writer per segment: no atomics
            const int tot = sh[0] + sh[1] + sh[2] + sh[3], c = sh[4] + sh[5] + sh[6] + sh[7];
            e.pub_lcnt[2 * seg] = tot;
            e.pub_lcnt[2 * seg + 1] = c;
            e.pub_lacc[2 * seg] += (unsigned long long)tot;
            e.pub_lacc[2 * seg + 1] += (unsigned long long)c;
        }
    }
    __syncthreads();
}

// By-products of a 3 x 3 or 1 x 1 edge, or of a residual skip, that its tiles leave to blocks of their own (publish_blocks of
// them): the source's list L (on the edge that carries it), the destination's compute list with its counts, the touched marks
// and the multiply-accumulate count.  A wave takes a segment of either list at a time, no barriers; a tile that made them itself had their loads ahead of
// its own and its loads behind their stores (memory operations of a wave complete in order): 2.0 us to the start of its K
// loop, now 1.3.  All loads of the two segments go out together, a row of the footprint is one unaligned word, and a mark is
// a byte store - a pixel has one owner, so nobody else writes its flag meanwhile - where an atomic OR went past the L2 of its
// XCD.  What bounds it is the number of instructions: one that needs the result of the one before it starts 8 cycles later.  The
// blocks of a 258 x 258 window were done 12.8 us into the launch, after its tiles, now 4.8; of a 66 x 66 window 6.3, now 2.5.
__device__ __forceinline__ void publish_edge(const EdgeDev& e, unsigned blk, unsigned nblk) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned long long below = (1ull << lane) - 1ull;
    const uint8_t* sflags = e.sflags;
    uint8_t* dflags = e.dflags;
    int *pub_list = e.pub_list, *pub_lcnt = e.pub_lcnt, *clist = e.clist, *ccnt = e.ccnt;
    unsigned long long *pub_lacc = e.pub_lacc, *cacc = e.cacc;
    int sH = e.sH, sW = e.sW, dH = e.dH, dW = e.dW, Hp = e.Hp, Wp = e.Wp, by0 = e.by0, bx0 = e.bx0, stride = e.stride, pad = e.pad, ks = e.k, up = e.up;
    read_now(sflags, dflags, pub_list, pub_lcnt, clist, ccnt, pub_lacc, cacc, sH, sW, dH, dW, Hp, Wp, by0, bx0, stride, pad, ks, up);
    const int HW = sH * sW, n = Hp * Wp;
    const int nsrc = pub_list ? (HW + kSegPixels - 1) / kSegPixels : 0, ndst = up ? 0 : (n + kSegPixels - 1) / kSegPixels;      // (an upsampling edge has no compute list, its tiles mark what they touch)
    const int units = nsrc > ndst ? nsrc : ndst;
    const float rw = rcp_of(Wp);
    // (a mark's byte outside the destination's view is read from beyond the end and its store dropped)
    const rsrc_t frs = make_rsrc(sflags, (unsigned)HW), wrs = taps3_rsrc(sflags, HW), mrs = make_rsrc(dflags, dflags ? (unsigned)(dH * dW) : 0u);
    constexpr unsigned kOutside = 0x80000000u;
    for (int s = (int)blk * 4 + wave; s < units; s += (int)nblk * 4) {
        const int p0 = s * kSegPixels + lane;
        unsigned f[4], df[4], at[4];                           // at: the pixel's flag in the destination
        Taps3 w[4];
        unsigned long long lsum[2] = {0, 0}, csum = 0;
        if (s < nsrc) {
#pragma unroll
            for (int k = 0; k < 4; ++k) f[k] = __builtin_amdgcn_raw_buffer_load_b8(frs, p0 + k * 64, 0, 0);
            if (lane == 0) { lsum[0] = pub_lacc[2 * s]; lsum[1] = pub_lacc[2 * s + 1]; }
        }
        if (s < ndst) {
            const int ry = (s * kSegPixels) / Wp, rx = s * kSegPixels - ry * Wp + lane;        // row of the segment's first pixel
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int x = rx + k * 64;                     // (fast_div below 2^24: a window has fewer columns)
                int q = (int)((float)x * rw);
                const int rem = x - q * Wp;
                q += (rem >= Wp ? 1 : 0) - (rem < 0 ? 1 : 0);
                const int cy = ry + q - by0, cx = x - q * Wp - bx0;
                const int iy = cy * stride - pad, ix = cx * stride - pad;
                const bool in = p0 + k * 64 < n;
                if (ks == 3) {
                    taps3_load(wrs, sH, sW, iy, ix, in, w[k]);
                } else {
                    w[k].cols = kFlagM;
                    w[k].w[1] = w[k].w[2] = 0;
                    w[k].w[0] = __builtin_amdgcn_raw_buffer_load_b8(frs, in && (unsigned)iy < (unsigned)sH && (unsigned)ix < (unsigned)sW ? iy * sW + ix : (int)kOutside, 0, 0);
                }
                at[k] = in && (unsigned)cy < (unsigned)dH && (unsigned)cx < (unsigned)dW ? (unsigned)(cy * dW + cx) : kOutside;
                df[k] = __builtin_amdgcn_raw_buffer_load_b8(mrs, (int)at[k], 0, 0);
            }
            if (lane == 0) csum = cacc[s];
        }
        if (s < nsrc) {
            int tot = 0, cand = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const unsigned long long bm = __ballot(f[k] & kFlagM);
                if (f[k] & kFlagM) pub_list[s * kSegPixels + tot + __popcll(bm & below)] = p0 + k * 64;
                tot += __popcll(bm);
                cand += __popcll(__ballot(f[k] & kFlagC));
            }
            if (lane == 0) {                                   // single writer per segment: no atomics
                pub_lcnt[2 * s] = tot;
                pub_lcnt[2 * s + 1] = cand;
                pub_lacc[2 * s] = lsum[0] + (unsigned long long)tot;
                pub_lacc[2 * s + 1] = lsum[1] + (unsigned long long)cand;
            }
        }
        if (s < ndst) {
            int tot = 0, taps = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                unsigned any = 0;
#pragma unroll
                for (int r = 0; r < 3; ++r) {
                    any |= w[k].w[r] & w[k].cols;
                    taps += __popc(w[k].w[r] & w[k].cols);
                }
                const unsigned long long b = __ballot(any != 0);
                if (any) {
                    clist[s * kSegPixels + tot + __popcll(b & below)] = p0 + k * 64;
                    __builtin_amdgcn_raw_buffer_store_b8((unsigned char)(df[k] | kFlagU), mrs, (int)at[k], 0, 0);     // outside: dropped
                }
                tot += __popcll(b);
            }
            taps = wave_sum(taps);
            if (lane == 0) {
                ccnt[s] = tot;
                cacc[s] = csum + (unsigned long long)tot;
                if (ks > 0) add_macs(e, taps, 0);              // (a residual skip multiplies nothing)
            }
        }
    }
}

// Readout within the last edge into an OUTPUT site: a tile writes f(P) of the entries it updates as it updates them, blocks of
// their own copy the pixels of the view that it leaves alone.  A launch of its own would wait for the tiles: 64 x 64
// convolution 15.0 -> 11.6 us, bottleneck 45.9 -> 43.8, five-layer network 60.8 -> 58.3.
template <typename T, int N>
__device__ __forceinline__ void write_out(T* out, int relu, size_t at, const T* v) {
    T o[N];
#pragma unroll
    for (int i = 0; i < N; ++i) o[i] = relu ? (T)fmaxf((float)v[i], 0.f) : v[i];
    __builtin_memcpy(out + at, o, N * sizeof(T));
}
// s_live: 256 bytes of LDS
template <typename T>
__device__ __forceinline__ void read_rest(const EdgeDev& e, unsigned blk, unsigned char* s_live) {
    constexpr int VEC = 16 / (int)sizeof(T);
    const int pieces = e.Cout / VEC, ppb = copy_pixels(pieces), first = (int)blk * ppb, tid = threadIdx.x;
    const int n = e.dH * e.dW - first < ppb ? e.dH * e.dW - first : ppb;
    const float rw = rcp_of(e.dW), rp = rcp_of(pieces);
    if (tid < n) {
        const int oy = div24(first + tid, e.dW, rw);
        const int ox = first + tid - oy * e.dW;
        s_live[tid] = e.up ? (e.sflags[(oy >> e.up) * e.sW + (ox >> e.up)] & kFlagM) != 0
                           : tap_mask(e, oy, ox) != 0;                   // (the view is where the convolution's output coordinates start)
    }
    __syncthreads();
    const T* const P = (const T*)e.P;
    T* const out = (T*)e.dY;
#pragma unroll 8
    for (int i = tid; i < n * pieces; i += 256) {
        const int p = div24(i, pieces, rp), c0 = (i - p * pieces) * VEC, pix = first + p;
        const int oy = div24(pix, e.dW, rw), ox = pix - oy * e.dW;
        T v[VEC];
        __builtin_memcpy(v, P + pdst_offset(e, oy + e.by0, ox + e.bx0) + c0, 16);
        if (!s_live[p]) write_out<T, VEC>(out, e.s_relu, (size_t)pix * e.Cout + c0, v);
    }
}

// What the blocks behind an edge's tiles do: [0, npub) publish, the rest read out.
template <typename T>
__device__ __forceinline__ void side_block(const EdgeDev& e, const TileGrid& g, unsigned blk, unsigned char* s_live) {
    if (blk < g.npub) publish_edge(e, blk, g.npub);
    else read_rest<T>(e, blk - g.npub, s_live);
}

}  // namespace mdcnn
