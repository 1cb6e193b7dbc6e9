// Convolution tile of the upsampling 1 x 1 fp16 edges of 64 n input channels.
#pragma once

#include "conv_device.h"

namespace mdcnn {

// ---------------------------------------------------------------------------
// A tile is 32 consecutive source pixels x 32 couts, and of the f x f pixels that each of them adds to four (all of them with
// f = 2): four times the blocks for the same sums, a few matrix instructions, and two pixels to a thread.  The four waves
// take every fourth 16 channels, operands straight from global memory; their sums are added through LDS in wave order.
//
// What bounds it: round trips.  An output pixel is made of one source pixel, so nothing has to be masked: a pixel that is not
// updated is multiplied and its result dropped.  Flags, rows, weights and pending values are all requested at once (early) where
// they are little; where they are more than the round trip takes, rows and pending values once the flags are there, of
// updated pixels only.
// HRNet-like 384 x 288 frame, pending values behind the flags / with them: 369 / 365 us, 8 videos 1001 / 991.
// ---------------------------------------------------------------------------
constexpr int kUpPx = 32, kUpCo = 32, kUpSum = kUpCo + 4, kUpSmem = 4 * kUpPx * kUpSum * 4;
__host__ __device__ inline int up_parts(int up) { return up > 1 ? 1 << (2 * up - 2) : 1; }     // blocks the f x f pixels are dealt to

// READ: the launch may read the destination out (EdgeDev::dY).  EARLY: everything is requested at once - code of its own, or each
// request waits for the flags that decide it in the other case.
template <bool READ, bool EARLY>
__device__ __forceinline__ void up_tile(const EdgeDev& e, unsigned blk, const TileGrid& g) {
    extern __shared__ __align__(16) unsigned char smem[];
    float* const sums = reinterpret_cast<float*>(smem);
    int sH = e.sH, sW = e.sW, Cin = e.Cin, Cout = e.Cout, Hp = e.Hp, Wp = e.Wp, by0 = e.by0, bx0 = e.bx0, p_oy = e.p_oy, p_ox = e.p_ox, up = e.up, dH = e.dH, dW = e.dW;
    const void *delta = e.delta, *w = e.w;
    const uint8_t* sflags = e.sflags;
    uint8_t* dflags = e.dflags;
    f16 *P = (f16*)e.P, *out_p = (f16*)e.dY;
    int NT = g.NT, MT = g.tiles_x, relu = e.s_relu;
    unsigned per_NT = g.per_NT, per_MT = g.per_tiles_x;
    read_now(sH, sW, Cin, Cout, Hp, Wp, by0, bx0, p_oy, p_ox, up, dH, dW, delta, w, sflags, dflags, P, NT, MT, per_NT, per_MT);
    P = in_global(P);
    if constexpr (READ) {
        read_now(out_p, relu);
        out_p = in_global(out_p);
    }
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r32 = lane & 31, kh = lane >> 5;
    const int t = by_reciprocal((int)blk, per_NT), n0 = ((int)blk - t * NT) * kUpCo;
    const int part = by_reciprocal(t, per_MT), p0 = (t - part * MT) * kUpPx;
    const int HW = sH * sW, f1 = (1 << up) - 1;
    constexpr unsigned kOutside = 0x80000000u;       // past the end of every tensor (the host checks that they are smaller than 2 GiB)
    const unsigned row = (unsigned)Cin * 2u;
    const rsrc_t frs = make_rsrc(sflags, (unsigned)HW), mrs = make_rsrc(dflags, dflags ? (unsigned)(dH * dW) : 0u);
    const rsrc_t drs = make_rsrc(delta, (unsigned)HW * row), wrs = make_rsrc(w, (unsigned)Cout * row);

    // what this thread adds to: eight couts of one of the four pixels, for two source pixels
    const int c8 = (tid & 3) * 8, at = part * 4 + (tid >> 2 & 3), a = at >> up, b = at & f1;
    const float rsw = rcp_of(sW);
    unsigned live[2], mark[2], df[2];
    f16* pp[2];
    f16x8 pold[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int px = p0 + (tid >> 4) + 16 * i, in = px < HW ? px : 0, cy = div24(in, sW, rsw), cx = in - cy * sW;
        const int oy = (cy << up) + a, ox = (cx << up) + b;
        live[i] = __builtin_amdgcn_raw_buffer_load_b8(frs, px < HW ? px : (int)kOutside, 0, 0);      // (outside: 0)
        mark[i] = px < HW && c8 == 0 && n0 == 0 ? (unsigned)(oy * dW + ox) : kOutside;             // (outside: dropped)
        pp[i] = P + ((size_t)wrapc(p_oy + by0 + oy, Hp) * Wp + wrapc(p_ox + bx0 + ox, Wp)) * Cout + n0 + c8;
    }
    const int px = p0 + r32;
    const unsigned mine = __builtin_amdgcn_raw_buffer_load_b8(frs, px < HW ? px : (int)kOutside, 0, 0);
    if (!EARLY && __ballot(mine & kFlagM) == 0) return;      // block-uniform
    const unsigned wl = (unsigned)(n0 + r32) * row + (unsigned)(wave * 32 + kh * 16);
    const unsigned bl = px < HW && (EARLY || (mine & kFlagM)) ? (unsigned)px * row + (unsigned)(wave * 32 + kh * 16) : kOutside;
    constexpr int D = 4;
    f16x8 fa[D], fb[D];
    const int nk = Cin / 64;                         // 16-channel blocks of a wave
    auto load = [&](int k, int d) {
        fa[d] = buf_load16(wrs, wl, (unsigned)k * 128u);
        fb[d] = buf_load16(drs, bl, (unsigned)k * 128u);
    };
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (d < nk) load(d, d);
    auto pending = [&](int i) {
        pold[i] = *reinterpret_cast<const f16x8*>(pp[i]);
        df[i] = __builtin_amdgcn_raw_buffer_load_b8(mrs, (int)mark[i], 0, 0);
    };
#pragma unroll
    for (int i = 0; i < 2; ++i)
        if (EARLY || (live[i] & kFlagM)) pending(i);         // (a tile's missing pixels read those of the first)
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    for (int k = 0; k < nk; k += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (k + d >= nk) break;
            acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[d], fb[d], acc, 0, 0, 0);
            if (k + d + D < nk) load(k + d + D, d);
        }
    }
    // register r: cout 8 * (r / 4) + 4 * kh + r % 4 of pixel r32
    float* dst = sums + (wave * kUpPx + r32) * kUpSum + 4 * kh;
#pragma unroll
    for (int q = 0; q < 4; ++q) *reinterpret_cast<float4*>(dst + 8 * q) = make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        if (!(live[i] & kFlagM)) continue;
        float v[8];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float* src = sums + (q * kUpPx + (tid >> 4) + 16 * i) * kUpSum + c8;
            const float4 v0 = *reinterpret_cast<const float4*>(src), v1 = *reinterpret_cast<const float4*>(src + 4);
            const float u[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
#pragma unroll
            for (int c = 0; c < 8; ++c) v[c] = q ? v[c] + u[c] : u[c];
        }
        f16x8 o = pold[i];
#pragma unroll
        for (int c = 0; c < 8; ++c) o[c] = (f16)((float)o[c] + v[c]);
        *reinterpret_cast<f16x8*>(pp[i]) = o;
        __builtin_amdgcn_raw_buffer_store_b8((unsigned char)(df[i] | kFlagU), mrs, (int)mark[i], 0, 0);
        if (READ && out_p) {                         // (the launch reads the site out)
            const int px2 = p0 + (tid >> 4) + 16 * i, cy = div24(px2, sW, rsw), cx = px2 - cy * sW;
            write_out<f16, 8>(out_p, relu, ((size_t)((cy << up) + a) * dW + (cx << up) + b) * Cout + n0 + c8, reinterpret_cast<const f16*>(&o));
        }
    }
    if (n0 == 0 && part == 0 && wave == 0) {         // statistics, once per tile
        const int n = __popcll(__ballot(lane < 32 && (mine & kFlagM)));
        if (lane == 0) add_macs(e, n, 0);
    }
}

template <bool READ>
__device__ __forceinline__ void up_body(const EdgeDev& e, unsigned blk, const TileGrid& g) {
    if (g.early) up_tile<READ, true>(e, blk, g);
    else up_tile<READ, false>(e, blk, g);
}

}  // namespace mdcnn
