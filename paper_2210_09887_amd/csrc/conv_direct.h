// Convolution tile straight from global memory to the matrix cores, fp16 or fp32.
#pragma once

#include "conv_device.h"

namespace mdcnn {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// A tile is 8 x 4 * TM window pixels x 32 * TN couts.  Nothing is staged: a lane
// of a wave holds pixel l % 32 (operand B) and cout l % 32 (operand A) and
// fetches 16 bytes of each per K block, lane half h the second 16 of the
// block's 32 bytes (16 fp16 or 8 fp32 channels).  The K blocks (tap-major) are
// dealt to the four waves in turn, two stages of D blocks in flight per wave, so
// a short layer is one round trip to memory; taps no pixel of the tile uses are
// passed over.  Rows of taps that miss the update mask read beyond the end of
// the tensor (zeros).  The four partial sums are added through LDS in wave
// order, whatever TM and TN: the bits of a layer do not depend on the tile.
//
// What bounds it: fp32 - the matrix instruction (256 cycles for the four of a K block
// against 64-100 of the L1 for its 2 KB of operands): 256 x 256 frame of the
// ResNet-18-style network in fp32 storage 80.6 ms -> 0.87 ms, its 128- to
// 512-channel layers ran as plain FMA with per-thread weights before.
// ---------------------------------------------------------------------------
template <typename T, int TM, int TN>
struct DirectCfg {
    static constexpr int TW = 8, TH = 4 * TM;        // window pixels of a tile
    static constexpr int PX = 32 * TM, CO = 32 * TN;
    static constexpr int LDC = CO + 4;               // partial-sum row, floats
    static constexpr int D = TM * TN >= 4 ? 3 : 4;   // K blocks per stage
    static constexpr int TPR = CO / 8;               // threads per pixel in the epilogue, 8 couts each
    static constexpr int RPP = 256 / TPR, NPASS = (PX + RPP - 1) / RPP;
    static constexpr int SMEM = 4 * PX * LDC * 4;
};

template <typename T> __device__ __forceinline__ f32x16 mfma_block(u32x4_t a, u32x4_t b, f32x16 c);
template <> __device__ __forceinline__ f32x16 mfma_block<f16>(u32x4_t a, u32x4_t b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}
template <> __device__ __forceinline__ f32x16 mfma_block<float>(u32x4_t a, u32x4_t b, f32x16 c) {
    const f32x4 x = __builtin_bit_cast(f32x4, a), y = __builtin_bit_cast(f32x4, b);
#pragma unroll
    for (int i = 0; i < 4; ++i) c = __builtin_amdgcn_mfma_f32_32x32x2f32(x[i], y[i], c, 0, 0, 0);
    return c;
}

// 8 stored values of one pixel: buffer loads / stores at a byte offset (beyond the tensor: zeros / dropped)
template <typename T> struct Px8;
template <> struct Px8<f16> {
    u32x4_t r;
    __device__ __forceinline__ void load(rsrc_t rs, unsigned off) { r = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, 0); }
    __device__ __forceinline__ void add_store(rsrc_t rs, unsigned off, const float* v) {
        f16x8 o = __builtin_bit_cast(f16x8, r);
#pragma unroll
        for (int q = 0; q < 8; ++q) o[q] = (f16)((float)o[q] + v[q]);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, o), rs, (int)off, 0, 0);
    }
};
template <> struct Px8<float> {
    u32x4_t r[2];
    __device__ __forceinline__ void load(rsrc_t rs, unsigned off) {
#pragma unroll
        for (int i = 0; i < 2; ++i) r[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(off + 16u * i), 0, 0);
    }
    __device__ __forceinline__ void add_store(rsrc_t rs, unsigned off, const float* v) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            f32x4 o = __builtin_bit_cast(f32x4, r[i]);
#pragma unroll
            for (int q = 0; q < 4; ++q) o[q] += v[4 * i + q];
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, o), rs, (int)(off + 16u * i), 0, 0);
        }
    }
};

constexpr unsigned kBeyond = 0x80000000u;            // a byte offset past every tensor (the host keeps them below 2 GiB)

// Tile with top left index-space pixel (y0, x0) - the padded window, or the source view of an upsampling edge - and first
// cout n0.  Block-uniform; called by all 256 threads; s_part: DirectCfg::SMEM bytes, s_vm: PX words.
template <typename T, int TM, int TN>
__device__ __forceinline__ void direct_tile(const EdgeDev& e, int y0, int x0, int n0, float* s_part, unsigned* s_vm) {
    using Cfg = DirectCfg<T, TM, TN>;
    constexpr int PX = Cfg::PX, LDC = Cfg::LDC, D = Cfg::D, TPR = Cfg::TPR, RPP = Cfg::RPP, NPASS = Cfg::NPASS;
    constexpr unsigned ES = sizeof(T);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r32 = lane & 31, h = lane >> 5;
    const int ih = e.up ? e.sH : e.Hp, iw = e.up ? e.sW : e.Wp;
    const int by = e.up ? 0 : e.by0, bx = e.up ? 0 : e.bx0;      // index space -> convolution output
    const unsigned row = (unsigned)e.Cin * ES;                   // bytes of a source pixel
    const rsrc_t drs = make_rsrc(e.delta, (unsigned)e.sH * (unsigned)e.sW * row);
    const rsrc_t prs = make_rsrc(e.P, (unsigned)e.Hp * (unsigned)e.Wp * (unsigned)e.Cout * ES);
    const bool packed = sizeof(T) == 2 && e.wp;
    const rsrc_t wrs = make_rsrc(packed ? e.wp : e.w, (unsigned)(e.k * e.k) * (unsigned)e.Cout * row);
    const int nkb = (int)(row / 32u), taps = e.k * e.k;

    unsigned vm[TM], om = 0;
    int bl[TM];                                                  // byte offset of the top left tap of this lane's pixel
#pragma unroll
    for (int t = 0; t < TM; ++t) {
        const int i = t * 32 + r32, iy = y0 + (i >> 3), ix = x0 + (i & 7);
        const int cy = iy - by, cx = ix - bx;
        const unsigned m = tap_mask(e, cy, cx);
        vm[t] = iy < ih && ix < iw ? m : 0u;
        bl[t] = ((cy * e.stride - e.pad) * e.sW + (cx * e.stride - e.pad)) * (int)row + 16 * h;
        om |= vm[t];
    }
#pragma unroll
    for (int o = 1; o < 32; o <<= 1) om |= __shfl_xor(om, o);    // both halves hold the same pixels
    om = (unsigned)__builtin_amdgcn_readfirstlane((int)om);
    if (om == 0) return;                                         // the four waves agree
    if (wave == 0 && h == 0) {
#pragma unroll
        for (int t = 0; t < TM; ++t) s_vm[t * 32 + r32] = vm[t];
    }

    // pending values of the epilogue (no upsampling: one pixel per entry) travel during the K loop
    const int c8 = (tid % TPR) * 8;
    Px8<T> pold[NPASS];
    unsigned poff[NPASS];
#pragma unroll
    for (int q = 0; q < NPASS; ++q) {
        const int i = tid / TPR + q * RPP, iy = y0 + (i >> 3), ix = x0 + (i & 7);
        const bool in = i < PX && iy < ih && ix < iw && n0 + c8 < e.Cout;
        const int wy = (iy << e.up) + (e.up ? e.by0 : 0), wx = (ix << e.up) + (e.up ? e.bx0 : 0);
        poff[q] = in ? (unsigned)(pdst_offset(e, wy, wx) + (size_t)(n0 + c8)) * ES : kBeyond;
        if (!e.up) pold[q].load(prs, poff[q]);
    }

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // this wave's K blocks: every fourth of (tap, block), inactive taps skipped
    int tap = 0, cb = wave;
    auto settle = [&]() {
        for (;;) {
            while (cb >= nkb) { cb -= nkb; ++tap; }
            if (tap >= taps || ((om >> tap) & 1u)) break;
            cb += 4;
        }
    };
    settle();
    // (a 16-cout layer has half a tile of weights)
    const unsigned wl = n0 + r32 >= e.Cout ? kBeyond : packed ? (unsigned)(r32 * 32 + 16 * h) : (unsigned)r32 * row + 16u * (unsigned)h;
    u32x4_t fa[2][D][TN], fb[2][D][TM];
    auto load = [&](int s) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const bool on = tap < taps;                          // wave-uniform
            const int jy = tap / e.k, jx = tap - jy * e.k;
            const int stepb = (jy * e.sW + jx) * (int)row + cb * 32;
            const unsigned stepa = packed ? ((unsigned)(tap * nkb + cb) * (unsigned)e.Cout + (unsigned)n0) * 32u
                                          : (unsigned)(tap * e.Cout + n0) * row + (unsigned)cb * 32u;
#pragma unroll
            for (int t = 0; t < TM; ++t) {
                const bool v = on && ((vm[t] >> (tap & 31)) & 1u);
                fb[s][d][t] = __builtin_amdgcn_raw_buffer_load_b128(drs, v ? bl[t] + stepb : (int)kBeyond, 0, 0);
            }
#pragma unroll
            for (int j = 0; j < TN; ++j)
                fa[s][d][j] = __builtin_amdgcn_raw_buffer_load_b128(wrs, (int)(on ? wl : kBeyond),
                                                                    on ? (int)(stepa + (packed ? 1024u : 32u * row) * (unsigned)j) : 0, 0);
            if (on) { cb += 4; settle(); }
        }
    };
    auto multiply = [&](int s) {
#pragma unroll
        for (int d = 0; d < D; ++d)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = mfma_block<T>(fa[s][d][j], fb[s][d][i], acc[i][j]);
    };
    load(0);
    for (;;) {
        const bool more = tap < taps;
        if (more) load(1);
        multiply(0);
        if (!more) break;
        const bool more2 = tap < taps;
        if (more2) load(0);
        multiply(1);
        if (!more2) break;
    }

    // partial sums -> LDS [wave][pixel][cout]; register r: cout 8 * (r / 4) + 4 * h + r % 4, pixel l % 32
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            float* dst = s_part + ((wave * PX) + i * 32 + r32) * LDC + j * 32 + 4 * h;
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *reinterpret_cast<float4*>(dst + 8 * g) =
                    make_float4(acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
        }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NPASS; ++q) {
        const int i = tid / TPR + q * RPP;
        if (i >= PX || s_vm[i] == 0 || poff[q] == kBeyond) continue;
        float v[8];
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float4 a = *reinterpret_cast<const float4*>(s_part + (w * PX + i) * LDC + c8);
            const float4 b = *reinterpret_cast<const float4*>(s_part + (w * PX + i) * LDC + c8 + 4);
            const float u[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = w ? v[k] + u[k] : u[k];
        }
        if (!e.up) {
            pold[q].add_store(prs, poff[q], v);
            continue;
        }
        const int iy = y0 + (i >> 3), ix = x0 + (i & 7), f = 1 << e.up;
        for (int a = 0; a < f; ++a)
            for (int b = 0; b < f; ++b) {
                const unsigned off = (unsigned)(pdst_offset(e, (iy << e.up) + e.by0 + a, (ix << e.up) + e.bx0 + b) + (size_t)(n0 + c8)) * ES;
                Px8<T> o;
                o.load(prs, off);
                o.add_store(prs, off, v);
            }
    }
    if (n0 == 0) {                                               // by the first cout tile: touched marks, statistics
        if (tid < PX && s_vm[tid]) {
            const int iy = y0 + (tid >> 3), ix = x0 + (tid & 7);
            mark_touched(e, (iy << e.up) + (e.up ? e.by0 : 0), (ix << e.up) + (e.up ? e.bx0 : 0));
        }
        if (wave == 0) {
            int n = 0;
#pragma unroll
            for (int t = 0; t < TM; ++t) n += __popc(vm[t]);
            n = wave_sum(n) >> 1;
            if (lane == 0) add_macs(e, n, 0);
        }
    }
}

// Writes list segment `seg` of the destination's compute list (256 consecutive window indices) and its counts.
__device__ __forceinline__ void publish_segment(const EdgeDev& e, int seg, int* sh) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int p = seg * kSegPixels + tid, wy = p / e.Wp, wx = p - wy * e.Wp;
    const bool in = p < e.Hp * e.Wp;
    const bool has = in && tap_mask(e, in ? wy - e.by0 : 0, in ? wx - e.bx0 : 0) != 0;
    const unsigned long long bal = __ballot(has);
    __syncthreads();                                             // sh is free
    if (lane == 0) sh[wave] = __popcll(bal);
    __syncthreads();
    int off = __popcll(bal & ((1ull << lane) - 1ull));
    for (int i = 0; i < wave; ++i) off += sh[i];
    if (has) e.clist[seg * kSegPixels + off] = p;
    if (tid == 0) {                                              // single writer per segment: no atomics
        const int tot = sh[0] + sh[1] + sh[2] + sh[3];
        e.ccnt[seg] = tot;
        e.cacc[seg] += (unsigned long long)tot;
    }
}

}  // namespace mdcnn
