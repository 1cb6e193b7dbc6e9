// Convolution tile of the fp32 layers on the matrix cores.
#pragma once

#include "conv_device.h"

namespace mdcnn {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// A tile is th x tw window pixels (th * tw <= 32) x 32 couts.  K runs over
// (32-channel chunk, active tap) steps; a step's weights [32][32] and delta rows
// [32][32] go global -> registers -> LDS, eight lanes to the 128 bytes of a row,
// and the four waves take 8 channels of the step each (v_mfma_f32_32x32x2_f32,
// lane half h the channels 4 h .. 4 h + 3 of the eight).  Two LDS stages, one
// barrier per step, two steps in flight in registers.  Taps no pixel of the tile
// uses are passed over; rows of taps that miss the update mask, channels past
// the last and couts past the last read beyond the end of the tensor (zeros).
// The four partial sums are added through LDS in wave order.
//
// What bounds it: the matrix instruction, 256 cycles of a wave per step.  A loop
// of nothing else takes 58 us for the products of 512 channels on a 34 x 34
// window (672 tiles, three to a compute unit), the launch 74 us.  Operands
// straight from global memory, as an earlier kernel took them, cost the L1 64
// cycles per load of a wave (four rows to a quad of lanes), twice the matrix
// instruction in all: that layer took 105 us.  128 channels on 66 x 66: 30.6 ->
// 22.7 us; 64 channels on 130 x 130, weights in LDS before: 35.4 -> 20.2 us;
// 256 x 256 frame of the ResNet-18-style network in fp32 storage 902 -> 666 us.
// Larger tiles (64 x 64: 95 us on the 512-channel layer, 27 us on the 64-channel
// one), more steps per barrier, deeper prefetch and operands read a step ahead
// were measured and are no faster.
// ---------------------------------------------------------------------------
constexpr int kF32Px = 32, kF32Co = 32;
constexpr int kF32Row = 36;                              // staged row, floats (32 channels + 16 bytes: no bank is hit twice)
constexpr int kF32Stage = (kF32Px + kF32Co) * kF32Row;   // floats of an LDS stage
constexpr int kF32Sum = kF32Co + 4;                      // partial-sum row, floats
constexpr int kF32Smem = (2 * kF32Stage > 4 * kF32Px * kF32Sum ? 2 * kF32Stage : 4 * kF32Px * kF32Sum);      // floats

// 8 stored values of one pixel: buffer loads / stores at a byte offset (beyond the tensor: zeros / dropped)
struct Px8 {
    u32x4_t r[2];
    __device__ __forceinline__ void load(rsrc_t rs, unsigned off) {
#pragma unroll
        for (int i = 0; i < 2; ++i) r[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(off + 16u * i), 0, 0);
    }
    __device__ __forceinline__ void add_store(rsrc_t rs, unsigned off, float* v, unsigned take = 0xffu) {      // take: bit k, v[k] is added; v becomes what is stored
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            f32x4 o = __builtin_bit_cast(f32x4, r[i]);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (take >> (4 * i + q) & 1u) o[q] += v[4 * i + q];
                v[4 * i + q] = o[q];
            }
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, o), rs, (int)(off + 16u * i), 0, 0);
        }
    }
};

constexpr unsigned kBeyond = 0x80000000u;            // a byte offset past every tensor (the host keeps them below 2 GiB)

// Tile with top left index-space pixel (y0, x0) - the padded window, or the source view of an upsampling edge - and first
// cout n0.  Block-uniform; called by all 256 threads; smem: kF32Smem floats, s_vm: kF32Px words, s_or: 4 words.  The caller
// has a barrier before the call.  take(wy, wx, c): which of the couts n0 + c .. n0 + c + 7 of a window pixel are wanted, a bit each
// (edges without upsampling); the others are left as they are.
struct AllCouts {
    __device__ __forceinline__ unsigned operator()(int, int, int) const { return 0xffu; }
};
template <typename Take = AllCouts>
__device__ __forceinline__ void f32_tile(const EdgeDev& e, int y0, int x0, int th, int tw, int n0, bool published, float* smem, unsigned* s_vm, unsigned* s_or,
                                         Take take = Take()) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r32 = lane & 31, h = lane >> 5;
    const int ih = e.up ? e.sH : e.Hp, iw = e.up ? e.sW : e.Wp;
    const int by = e.up ? 0 : e.by0, bx = e.up ? 0 : e.bx0;      // index space -> convolution output
    const unsigned row = (unsigned)e.Cin * 4u;                   // bytes of a source pixel
    const rsrc_t drs = make_rsrc(e.delta, (unsigned)e.sH * (unsigned)e.sW * row);
    const rsrc_t prs = make_rsrc(e.P, (unsigned)e.Hp * (unsigned)e.Wp * (unsigned)e.Cout * 4u);
    const rsrc_t wrs = make_rsrc(e.w, (unsigned)(e.k * e.k) * (unsigned)e.Cout * row);
    const float rtw = rcp_of(tw);
    auto pixel = [&](int i, int& iy, int& ix) {                  // pixel i of the tile; false: none
        const int ly = fast_div(i, tw, rtw);
        iy = y0 + ly;
        ix = x0 + i - ly * tw;
        return ly < th && iy < ih && ix < iw;
    };

    // the rows this thread stages: pixel and cout tid / 8, 16-byte piece tid % 8 of the chunk
    const int prow = tid >> 3, piece = tid & 7;
    int py, px;
    const bool pin = pixel(prow, py, px);
    const int cy = py - by, cx = px - bx;
    unsigned vm = tap_mask(e, pin ? cy : 0, pin ? cx : 0);
    if (!pin) vm = 0u;
    const int bl = ((cy * e.stride - e.pad) * e.sW + (cx * e.stride - e.pad)) * (int)row + 16 * piece;     // the pixel's top left tap
    const unsigned wl = n0 + prow < e.Cout ? (unsigned)(n0 + prow) * row + 16u * (unsigned)piece : kBeyond;
    if (piece == 0) s_vm[prow] = vm;
    unsigned om = vm;
#pragma unroll
    for (int o = 8; o < 64; o <<= 1) om |= __shfl_xor(om, o);
    if (lane == 0) s_or[wave] = om;
    __syncthreads();
    om = (unsigned)__builtin_amdgcn_readfirstlane((int)(s_or[0] | s_or[1] | s_or[2] | s_or[3]));
    if (om == 0) return;                                         // block-uniform

    const int nc = (e.Cin + 31) / 32, steps = nc * __popc(om);
    int c = 0;                                                   // next step to fetch: chunk, taps left in it
    unsigned left = om;
    u32x4_t ra[2], rb[2];
    const int kinv = 65536 / e.k + 1;                            // tap / k == tap * kinv >> 16 for tap < 25
    const int line = (e.sW - e.k) * (int)row;                    // tap (jy, jx): jy source rows and jx pixels on
    const unsigned wtap = (unsigned)e.Cout * row;
    auto fetch = [&](int g) {                                    // past the last step: zeros
        // dead operands get bit 31 of their offset set, which is past every tensor: a condition here becomes a branch, and
        // the loads of its two sides wait for everything in flight
        const unsigned off = c < nc && c * 32 + piece * 4 < e.Cin ? 0u : kBeyond;
        const int tap = __builtin_ctz(left);
        left &= left - 1;
        const int jy = tap * kinv >> 16;
        const int stepb = jy * line + tap * (int)row + c * 128;
        const unsigned stepa = (unsigned)tap * wtap + (unsigned)c * 128u;
        const unsigned dead = (~vm >> tap) << 31;
        ra[g] = __builtin_amdgcn_raw_buffer_load_b128(wrs, (int)(wl | off), (int)stepa, 0);
        rb[g] = __builtin_amdgcn_raw_buffer_load_b128(drs, (int)((unsigned)(bl + stepb) | dead | off), 0, 0);
        if (left == 0) { left = om; ++c; }
    };
    auto stage = [&](int g) {                                    // a step's registers -> LDS stage of the same number
        float* dst = smem + g * kF32Stage + prow * kF32Row + piece * 4;
        *reinterpret_cast<u32x4_t*>(dst) = ra[g];
        *reinterpret_cast<u32x4_t*>(dst + kF32Co * kF32Row) = rb[g];
    };
    fetch(0);
    fetch(1);

    // pending values of the epilogue (eight couts of a pixel per thread; no upsampling: one pixel per entry) travel during the K loop
    const int c8 = (tid % 4) * 8, pi = tid / 4;
    int wy, wx;
    const bool mine = pixel(pi, wy, wx) && pi < kF32Px && n0 + c8 < e.Cout;
    wy = (wy << e.up) + (e.up ? e.by0 : 0);
    wx = (wx << e.up) + (e.up ? e.bx0 : 0);
    const unsigned poff = mine ? (unsigned)(pdst_offset(e, wy, wx) + (size_t)(n0 + c8)) * 4u : kBeyond;
    Px8 pold;
    if (!e.up) pold.load(prs, poff);

    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    stage(0);
    fetch(0);
    __syncthreads();
    for (int s = 0; s < steps; s += 2) {                         // (an odd last step is followed by one of zeros)
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            const float* src = smem + g * kF32Stage + r32 * kF32Row + wave * 8 + 4 * h;
            const f32x4 fa = *reinterpret_cast<const f32x4*>(src);
            const f32x4 fb = *reinterpret_cast<const f32x4*>(src + kF32Co * kF32Row);
            stage(1 - g);                                        // (read before the last barrier)
            fetch(1 - g);
#pragma unroll
            for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i], fb[i], acc, 0, 0, 0);
            __syncthreads();
        }
    }

    // partial sums -> LDS [wave][pixel][cout]; register r: cout 8 * (r / 4) + 4 * h + r % 4, pixel l % 32
    float* dst = smem + (wave * kF32Px + r32) * kF32Sum + 4 * h;
#pragma unroll
    for (int g = 0; g < 4; ++g)
        *reinterpret_cast<float4*>(dst + 8 * g) = make_float4(acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]);
    __syncthreads();
    if (mine && s_vm[pi]) {
        float v[8];
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float4 a = *reinterpret_cast<const float4*>(smem + (w * kF32Px + pi) * kF32Sum + c8);
            const float4 b = *reinterpret_cast<const float4*>(smem + (w * kF32Px + pi) * kF32Sum + c8 + 4);
            const float u[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = w ? v[k] + u[k] : u[k];
        }
        if (!e.up) {
            const unsigned want = take(wy, wx, c8);
            if (want) pold.add_store(prs, poff, v, want);
            if (want && e.dY) {                                        // (the launch reads the site out)
                const int oy = wy - e.by0, ox = wx - e.bx0;
                if ((unsigned)oy < (unsigned)e.dH && (unsigned)ox < (unsigned)e.dW)
                    write_out<float, 8>((float*)e.dY, e.s_relu, ((size_t)oy * e.dW + ox) * e.Cout + n0 + c8, v);
            }
        } else {
            const int f = 1 << e.up;
            for (int a = 0; a < f; ++a)
                for (int b = 0; b < f; ++b) {
                    const unsigned off = (unsigned)(pdst_offset(e, wy + a, wx + b) + (size_t)(n0 + c8)) * 4u;
                    Px8 o;
                    o.load(prs, off);
                    float s[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) s[k] = v[k];
                    o.add_store(prs, off, s);
                }
        }
    }
    if (n0 == 0 && wave == 0 && !published) {                    // by the first cout tile: touched marks, statistics
        const unsigned m = tid < kF32Px ? s_vm[tid] : 0u;
        if (m) {
            int iy, ix;
            pixel(tid, iy, ix);
            mark_touched(e, (iy << e.up) + (e.up ? e.by0 : 0), (ix << e.up) + (e.up ? e.bx0 : 0));
        }
        const int n = wave_sum(__popc(m));
        if (lane == 0) add_macs(e, n, 0);
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
