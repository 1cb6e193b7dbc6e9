// Convolution tile of the 3 x 3 fp32 layers of 64 n input channels: products on the bf16 matrix instruction.
#pragma once

#include "conv_f32.h"

namespace mdcnn {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));

constexpr int split_rows(int tm) { return tm == 1 ? 4 : tm == 2 ? 7 : 9; }      // staged rows of a tile of tm row tiles

// ---------------------------------------------------------------------------
// A tile is a th x tw rectangle of the padded window (tw <= 14, th * tw <= 32 TM) x 32 couts; its live pixels are ranked as
// those of conv_rect.h and TM row tiles of 32 of them multiplied.  An fp32 value is the exact sum of three bf16, each the rest
// rounded to the nearest (Henry, Tang, Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype For Higher-Precision
// Computations", 2019), and a product six of the nine products of their parts, each exact in the fp32 accumulators of
// v_mfma_f32_32x32x16_bf16: 192 cycles for 16 channels where v_mfma_f32_32x32x2_f32 takes 512.  Those of the leading parts have
// accumulators of their own, a rounding per 16 channels instead of one per channel: against 64 bits, 64 to 512 channels of normal
// and rectified values, 0.8e-7 to 2.0e-7 of the result, with fp32 products 1.6e-7 to 6.0e-7.  The three products left out are 2^-24 of
// the whole one at most, half a unit of its last place: a sum of ONE product is off by 2.59e-8 (root mean square; worst seen 0.9 units), with
// fp32 products 2.53e-8 (0.5); of two 3.54e-8 against 3.58e-8, of 16 4.9e-8 against 5.8e-8.  Two products more would mend the first at 500
// us for 470 of a 256 x 256 frame of the ResNet-18-style network.
//
// The footprint of the tile is fetched per 64-channel chunk, split once for its nine taps and kept in LDS, part by part, in rows
// of 16 pixels.  A pixel takes 144 bytes and a row is further on by as many 16-byte steps as its tw entries have taken, so
// that the 16 lanes whose reads go together, with 16 consecutive entries (entry_of_lane), are on banks of their own while all
// pixels are live.  Each of the four waves takes 16 channels of a chunk: it fetches the weights of a tap three steps ahead,
// splits them, and passes them between its lanes through LDS of its own, which takes no barrier, the LDS operations of a wave
// being in order.  The four partial sums are added through LDS in wave order, so the tile does not change a result.
//
// A part of an infinity or NaN is none: sums that are not finite in either of two passes are made with products in fp32 (f32_tile), and they alone, from
// runs of 16 window columns that every tile has in common - a value is that of its own operands, whatever shares the tile, and a
// video of a batch, where tiles are of another size, gives the bits it gives alone.
//
// What bounds it: the issue of instructions, about 83 of a step beside its 6 TM products, 52 of them the split of the weights,
// at 4.6 cycles each - 0.34 us a step with two row tiles, whether one block is on a compute unit or two share it.  Counted on 512 -> 512, three
// row tiles, one wave to a SIMD: vector instructions are issued 38 % of a wave's time, the matrix pipe is busy 41 %, the two hardly at once; 24 %
// are waits.  Chains of
// one layer, all pixels updated, us a frame (10 of them not this launch), before (k_conv_f32) and now: 512 -> 512 on 32 x 32 84.9 and
// 58.0, 256 -> 256 34.1 and 24.7, 128 -> 128 on 64 x 64 28.5 and 22.8, 64 -> 64 on 128 x 128 27.9 and 25.4, on 256 x 256
// 82.7 and 65.9.  Stride 2, with a footprint four times the tile, was no faster than k_conv_f32 (64 -> 128: 23.4 and 21.3).  Not
// faster either: weights fetched nine steps ahead, other orders of the instructions of a step.  The multiplications by powers of two
// of the split are within the noise where they are (512 -> 512 47.8 and 48.4, 256 -> 256 23.0 and 22.4, in another run).
// ---------------------------------------------------------------------------
template <int TM_>
struct SplitCfg {
    static constexpr int TM = TM_, M = 32 * TM;
    static constexpr int MINB = 4 - TM;              // tiles to a compute unit
    static constexpr int NBUF = MINB == 1 ? 2 : 1;   // chunks of rows in LDS, steps whose operands are in registers
    static constexpr int ROWS = split_rows(TM);
    static constexpr int PXP = 144;                  // bytes from pixel to pixel: 64 bf16 and 16 more
    static constexpr int PLANE = ROWS * (16 * PXP + 240);
    static constexpr int WP = 48, WPLANE = 32 * WP;  // a wave's weights: bytes from cout to cout, from part to part
    static constexpr int SUMS = 4 * M * kF32Sum * 4;
    static constexpr int ROW_BYTES = 3 * NBUF * PLANE > SUMS ? 3 * NBUF * PLANE : SUMS;
    static constexpr int LEFT = ROW_BYTES + 4 * 3 * WPLANE + M * 4;
    static constexpr int SMEM = LEFT + M * 4 + ROWS * 4;
    static_assert(ROW_BYTES >= kF32Smem * 4 + kF32Px * 4 + 16, "the tile of conv_f32.h in the same place");
    static_assert(SMEM * MINB <= 160 * 1024);
};

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned pack_bf16(float a, float b) {
    return __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2{a, b}), bf16x2));
}
// x scale = p[0] + p[1] + p[2] (each the rest rounded to the nearest bf16), exactly if x scale is below 2^128 and x's last place, scaled,
// 2^-126 or above: the matrix instruction takes a subnormal operand for zero
__device__ __forceinline__ void split_bf16(u32x4_t raw, float scale, u32x2_t* p) {
    const f32x4 x = __builtin_bit_cast(f32x4, raw);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        float a = x[2 * i] * scale, b = x[2 * i + 1] * scale;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const unsigned h = pack_bf16(a, b);
            p[q][i] = h;
            if (q < 2) {
                a -= __builtin_bit_cast(float, h << 16);
                b -= __builtin_bit_cast(float, h & 0xffff0000u);
            }
        }
    }
}

__device__ __forceinline__ bool finite(float x) { return __builtin_fabsf(x) <= 3.4028234e38f; }

// Which of 32 entries a lane has: the 16 lanes whose 16-byte LDS reads go together (0-3, 12-15, 20-27; the others) have consecutive ones.
__device__ __forceinline__ int entry_of_lane(int l) {
    const bool second = (l >= 4 && l < 12) || (l >= 16 && l < 20) || l >= 28;
    return second ? (l < 12 ? l + 12 : l < 20 ? l + 8 : l) : (l < 4 ? l : l < 16 ? l - 8 : l - 12);
}

// Weights and delta rows are multiplied by powers of two first, so that the parts of the smallest values are normal numbers: 2^-149
// becomes 2^-125 (as they were, frames of 1e-36 came out 2^-15 off and weights of 1e-36 2^-11, subnormal ones as zeros; fp32 products are
// 2^-22.5 off there as everywhere, these now 2^-23.7).  What that makes too large, rows from 2^104 or sums from 2^80 on, comes out not
// finite and is made again with rows divided by 2^40.  Rows below 2^-62 lose up to 2^-86 by that, products with the largest weight that
// this pass holds 2^18: far below the roundings of a sum of 2^64.  Smaller ones, where weights of zero meet the large rows, are left to fp32.
constexpr float kSplitWeights = 0x1p24f, kSplitRows = 0x1p24f, kSplitRowsLarge = 0x1p-40f, kSplitLeast = 0x1p64f * kSplitWeights * kSplitRowsLarge;

// The sums of a tile; false: that was all of them.  again: those that are not finite once more (left: this thread's, eight bits to an entry),
// and which are not even then, or too small for this pass, goes to s_left.
template <typename Cfg>
__device__ __forceinline__ bool split_pass(const EdgeDev& e, unsigned blk, const TileGrid& g, bool again, unsigned& left) {
    constexpr int TM = Cfg::TM, M = Cfg::M, ROWS = Cfg::ROWS, PXP = Cfg::PXP, PLANE = Cfg::PLANE, WP = Cfg::WP, WPLANE = Cfg::WPLANE, NBUF = Cfg::NBUF, R = 3;
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* const s_w = smem + Cfg::ROW_BYTES;
    int* const s_ent = reinterpret_cast<int*>(s_w + 4 * 3 * WPLANE);        // entry -> ly << 4 | lx
    unsigned char* const s_left = smem + Cfg::LEFT;                            // sums still to be made: [pixel of the tile][cout / 8], a bit each
    unsigned char* const s_mask = s_left + 4 * M;                              // updated pixels of a staged row, four bits a wave
    int Hp = e.Hp, Wp = e.Wp, sH = e.sH, sW = e.sW, Cin = e.Cin, Cout = e.Cout, by0 = e.by0, bx0 = e.bx0, pad = e.pad;
    int NT = g.NT, th = g.p0, tw = g.p1, tiles_x = g.tiles_x;
    unsigned per_NT = g.per_NT, per_tiles_x = g.per_tiles_x;
    read_now(Hp, Wp, sH, sW, Cin, Cout, by0, bx0, pad, NT, th, tw, tiles_x, per_NT, per_tiles_x);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r32 = lane & 31, h = lane >> 5, e32 = entry_of_lane(r32);
    const int nchunks = Cin / 64;
    const float up = again ? kSplitRowsLarge : kSplitRows, down = again ? 1 / (kSplitWeights * kSplitRowsLarge) : 1 / (kSplitWeights * kSplitRows);
    const int pitch = 16 * (PXP + (9 * tw & 15));
    const unsigned row = (unsigned)Cin * 4u;         // bytes of a source pixel
    const rsrc_t drs = make_rsrc(e.delta, (unsigned)sH * (unsigned)sW * row);
    const rsrc_t frs = make_rsrc(e.sflags, (unsigned)sH * (unsigned)sW);
    const rsrc_t prs = make_rsrc(e.P, (unsigned)Hp * (unsigned)Wp * (unsigned)Cout * 4u);
    const rsrc_t wrs = make_rsrc(e.w, 9u * (unsigned)Cout * row);
    const int mt = by_reciprocal((int)blk, per_NT), nt = (int)blk - mt * NT, n0 = nt * 32;
    const int ty = by_reciprocal(mt, per_tiles_x), tx = mt - ty * tiles_x;
    const int wy0 = ty * th, wx0 = tx * tw;
    const int nty = wy0 + th < Hp ? th : Hp - wy0, ntx = wx0 + tw < Wp ? tw : Wp - wx0;
    // staged by this thread: pixel sx of every row, 16 bytes of its chunk
    const int sx = tid >> 4, piece = tid & 15;
    const int iy = wy0 - by0 - pad, ix = wx0 - bx0 - pad + sx;
    const bool xin = sx < ntx + 2 && ix >= 0 && ix < sW;
    const unsigned pix = (unsigned)(iy * sW + ix);
    unsigned fl[ROWS];
#pragma unroll
    for (int j = 0; j < ROWS; ++j) {
        const bool in = xin && j < nty + 2 && iy + j >= 0 && iy + j < sH;
        fl[j] = __builtin_amdgcn_raw_buffer_load_b8(frs, (int)(in ? pix + (unsigned)(j * sW) : kBeyond), 0, 0);      // (outside: 0)
    }
    // weights of a step: 32 couts x this wave's 16 channels, four lanes to a cout's 64 bytes
    const unsigned tap_stride = (unsigned)Cout * row;
    const unsigned wlane = (unsigned)(n0 + (lane >> 2)) * row + (unsigned)(wave * 64 + (lane & 3) * 16);
    u32x4_t rw[R][2];
    auto fetch_w = [&](int slot, int c, int tap) {
        const unsigned src = (unsigned)tap * tap_stride + (unsigned)c * 256u;
        rw[slot][0] = __builtin_amdgcn_raw_buffer_load_b128(wrs, (int)wlane, (int)src, 0);
        rw[slot][1] = __builtin_amdgcn_raw_buffer_load_b128(wrs, (int)wlane, (int)(src + 16u * row), 0);
    };
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < R; ++i) fetch_w(i, 0, i);
    __builtin_amdgcn_sched_barrier(0);
    unsigned src[ROWS];
    u32x4_t raw[ROWS];
#pragma unroll
    for (int j = 0; j < ROWS; ++j) src[j] = ((pix + (unsigned)(j * sW)) * row + (unsigned)piece * 16u) | (~fl[j] >> 2) << 31;      // kFlagM == 4
    auto fetch_rows = [&](int c) {
#pragma unroll
        for (int j = 0; j < ROWS; ++j) raw[j] = __builtin_amdgcn_raw_buffer_load_b128(drs, (int)src[j], c * 256, 0);
    };
    fetch_rows(0);
    unsigned char bits[ROWS];
#pragma unroll
    for (int j = 0; j < ROWS; ++j) {
        const unsigned long long b = __ballot(fl[j] & kFlagM) & 0x0001000100010001ull;                 // sixteen lanes to a pixel
        bits[j] = (unsigned char)(b | b >> 15 | b >> 30 | b >> 45) & 15;
    }
    if (lane == 0) {
#pragma unroll
        for (int j = 0; j < ROWS; ++j) s_mask[4 * j + wave] = bits[j];
    }
    __syncthreads();
    // the live pixels of the tile, ranked row by row: lane l of every wave has row l
    int any = 0;
    if (lane < nty) {
        const unsigned* r = reinterpret_cast<const unsigned*>(s_mask) + lane;
        const unsigned v = r[0] | r[1] | r[2];
        int m = (int)((v & 0xfu) | (v >> 4 & 0xf0u) | (v >> 8 & 0xf00u) | (v >> 12 & 0xf000u));
        m = m | m >> 1 | m >> 2;
        any = m & ((1 << ntx) - 1);
    }
    int upto = __popc(any);
    upto += __builtin_amdgcn_update_dpp(0, upto, 0x111, 0xf, 0xf, false);      // sums within 16 lanes (a tile has no more rows)
    upto += __builtin_amdgcn_update_dpp(0, upto, 0x112, 0xf, 0xf, false);
    upto += __builtin_amdgcn_update_dpp(0, upto, 0x114, 0xf, 0xf, false);
    upto += __builtin_amdgcn_update_dpp(0, upto, 0x118, 0xf, 0xf, false);
    const int tot = __builtin_amdgcn_readlane(upto, 15);
    if (tot == 0) return false;                       // block-uniform
    if (tid < M) {
        const int ly = fast_div(tid, tw, rcp_of(tw)), lx = tid - ly * tw;
        const int a = __shfl(any, ly), before = __shfl(upto, ly) - __popc(a);
        if (ly < nty && (a >> lx & 1)) s_ent[before + __popc(a & ((1 << lx) - 1))] = ly << 4 | lx;
    }
    auto store_row = [&](int j, int buf) {
        u32x2_t p[3];
        split_bf16(raw[j], up, p);
#pragma unroll
        for (int q = 0; q < 3; ++q) *reinterpret_cast<u32x2_t*>(smem + (buf * 3 + q) * PLANE + j * pitch + sx * PXP + piece * 8) = p[q];
    };
    auto store_rows = [&] {
#pragma unroll
        for (int j = 0; j < ROWS; ++j) store_row(j, 0);
    };
    unsigned char* const my_w = s_w + wave * 3 * WPLANE;
    auto store_w = [&](int slot) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            u32x2_t p[3];
            asm volatile("" : "+v"(rw[slot][i]));      // (or the multiplication goes up to where the weights are asked for, and waits: 490 us for 470)
            split_bf16(rw[slot][i], kSplitWeights, p);
#pragma unroll
            for (int q = 0; q < 3; ++q) *reinterpret_cast<u32x2_t*>(my_w + q * WPLANE + (i * 16 + (lane >> 2)) * WP + (lane & 3) * 8) = p[q];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // (read by the other lanes of the wave)
    };
    // refill of the slot whose weights, those of step i of chunk c, have just been stored
    // (past the last chunk: its own again, not used)
    auto refill = [&](int slot, int c, int i) {
        const int at = i + R < 9 ? c : c + 1;
        fetch_w(slot, at < nchunks ? at : nchunks - 1, (i + R) % 9);
    };
    store_w(0);
    refill(0, 0, 0);
    store_rows();
    __syncthreads();
    const int nrt = (tot + 31) >> 5;                  // live row tiles
    int off[TM][3];                                   // this lane's operand at taps (dy, 0)
#pragma unroll
    for (int t = 0; t < TM; ++t) {
        const int r = t * 32 + e32, ent = s_ent[r < tot ? r : 0];
#pragma unroll
        for (int dy = 0; dy < 3; ++dy) off[t][dy] = ((ent >> 4) + dy) * pitch + (ent & 15) * PXP + (2 * wave + h) * 16;
    }
    const unsigned char* const wsrc = my_w + r32 * WP + h * 16;

    f32x16 acc[TM], low[TM];                          // products of the leading parts; all others
#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = low[t][r] = 0.f;

    auto kloop = [&](auto lc) {
        constexpr int L = decltype(lc)::value;
        bf16x8 fw[NBUF][3], fr[NBUF][3][L];
        auto chunk = [&](auto par, int c) {
            constexpr int PAR = decltype(par)::value;
            auto operands = [&](int slot, int i) {
#pragma unroll
                for (int q = 0; q < 3; ++q) fw[slot][q] = *reinterpret_cast<const bf16x8*>(wsrc + q * WPLANE);
#pragma unroll
                for (int q = 0; q < 3; ++q)
#pragma unroll
                    for (int t = 0; t < L; ++t)
                        fr[slot][q][t] = *reinterpret_cast<const bf16x8*>(smem + ((PAR % NBUF) * 3 + q) * PLANE + (i % 3) * PXP + off[t][i / 3]);
            };
            const bool more = c + 1 < nchunks;
            if (more) fetch_rows(c + 1);
            if constexpr (NBUF == 2) operands(PAR, 0);
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                const int slot = NBUF == 2 ? (PAR + i) & 1 : 0;
                if constexpr (NBUF == 1) operands(0, i);
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                store_w((i + 1) % R);                  // (the wave's own weights: its LDS operations are in order)
                refill((i + 1) % R, i < 8 ? c : c + 1, (i + 1) % 9);
                if (NBUF == 2 && i < 8) operands(slot ^ 1, i + 1);
#pragma unroll
                for (int u = 0; u < 6; ++u) {
                    constexpr int qw[6] = {0, 2, 0, 1, 1, 0}, qr[6] = {0, 0, 2, 1, 0, 1};
#pragma unroll
                    for (int t = 0; t < L; ++t) {
                        f32x16& to = u ? low[t] : acc[t];
                        to = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[slot][qw[u]], fr[slot][qr[u]][t], to, 0, 0, 0);
                    }
                }
                if constexpr (TM == 3) {               // four others between two products: pays for the multiplications here, 465 -> 458 us a 256 x 256 frame (fewer row tiles: slower)
#pragma unroll
                    for (int u = 0; u < 6 * L; ++u) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
                    }
                }
                if constexpr (NBUF == 2) {
                    if (more && i >= 3) {
#pragma unroll
                        for (int j = 2 * (i - 3); j < 2 * (i - 2) && j < ROWS; ++j) store_row(j, PAR ^ 1);
                    }
                }
            }
            if (more) {
                __syncthreads();                       // the staged rows have been read
                if constexpr (NBUF == 1) {
                    store_rows();
                    __syncthreads();
                }
            }
        };
        for (int c = 0; c < nchunks; c += 2) {
            chunk(std::integral_constant<int, 0>{}, c);
            if (c + 1 < nchunks) chunk(std::integral_constant<int, 1>{}, c + 1);
        }
#pragma unroll
        for (int t = 0; t < L; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[t][r] += low[t][r];
    };
    if (TM >= 3 && nrt == 3) kloop(std::integral_constant<int, TM >= 3 ? 3 : TM>{});
    else if (TM >= 2 && nrt == 2) kloop(std::integral_constant<int, TM >= 2 ? 2 : TM>{});
    else kloop(std::integral_constant<int, 1>{});

    // P <- P + sum, four threads to an entry
    constexpr int NPASS = (M + 63) / 64;
    const int c8 = (tid & 3) * 8;
    Px8 pold[NPASS];
    unsigned poff[NPASS];
#pragma unroll
    for (int t = 0; t < NPASS; ++t) {
        const int at = t * 64 + (tid >> 2), en = s_ent[at < tot ? at : 0];
        poff[t] = at < tot ? (unsigned)(pdst_offset(e, wy0 + (en >> 4), wx0 + (en & 15)) + (size_t)(n0 + c8)) * 4u : kBeyond;
        pold[t].load(prs, poff[t]);
    }
    float* const sums = reinterpret_cast<float*>(smem);
    __syncthreads();                                  // the staged rows have been read
#pragma unroll
    for (int t = 0; t < TM; ++t) {
        if (t >= nrt) break;
        float* dst = sums + (wave * M + t * 32 + e32) * kF32Sum + 4 * h;       // register r: cout 8 * (r / 4) + 4 * h + r % 4
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<float4*>(dst + 8 * q) = make_float4(acc[t][4 * q], acc[t][4 * q + 1], acc[t][4 * q + 2], acc[t][4 * q + 3]);
    }
    __syncthreads();
    float v[NPASS][8];
    bool bad = false;
#pragma unroll
    for (int t = 0; t < NPASS; ++t) {
        const int at = t * 64 + (tid >> 2);
        if (at >= tot) continue;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float4 a = *reinterpret_cast<const float4*>(sums + (w * M + at) * kF32Sum + c8);
            const float4 b = *reinterpret_cast<const float4*>(sums + (w * M + at) * kF32Sum + c8 + 4);
            const float u[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
            for (int k = 0; k < 8; ++k) v[t][k] = w ? v[t][k] + u[k] : u[k];
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) bad |= !finite(v[t][k]);
    }
    auto finish = [&](auto some) {                    // some: not all of them, or not all are as they should be
#pragma unroll
        for (int t = 0; t < NPASS; ++t) {
            const int at = t * 64 + (tid >> 2);
            if (at >= tot) continue;
            unsigned done = 0xffu;
            if constexpr (decltype(some)::value) {
                done = 0;
#pragma unroll
                for (int k = 0; k < 8; ++k) done |= finite(v[t][k]) && (!again || __builtin_fabsf(v[t][k]) >= kSplitLeast) ? 1u << k : 0u;
                done &= left >> (8 * t);
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) v[t][k] *= down;
            pold[t].add_store(prs, poff[t], v[t], done);
            const int en = s_ent[at], ly = en >> 4, lx = en & 15;
            if (e.dY) {                               // (the launch reads the site out)
                const int oy = wy0 + ly - by0, ox = wx0 + lx - bx0;
                if ((unsigned)oy < (unsigned)e.dH && (unsigned)ox < (unsigned)e.dW)
                    write_out<float, 8>((float*)e.dY, e.s_relu, ((size_t)oy * e.dW + ox) * e.Cout + n0 + c8, v[t]);
            }
            if constexpr (decltype(some)::value) {
                left &= ~(done << (8 * t));
                if (again) s_left[(ly * tw + lx) * 4 + (tid & 3)] = (unsigned char)(left >> (8 * t));
            }
        }
    };
    if (!again && !__syncthreads_or(bad)) {
        finish(std::false_type{});
        return false;
    }
    if (!again) {
#pragma unroll
        for (int t = 0; t < NPASS; ++t) left |= t * 64 + (tid >> 2) < tot ? 0xffu << (8 * t) : 0u;
    } else {
        if (tid < M) reinterpret_cast<int*>(s_left)[tid] = 0;
        __syncthreads();
    }
    finish(std::true_type{});
    return __syncthreads_or(left != 0);
}

template <typename Cfg>
__device__ __forceinline__ void split_tile(const EdgeDev& e, unsigned blk, const TileGrid& g) {
    unsigned left = 0;
#pragma unroll 1
    for (int again = 0; again < 2; ++again)
        if (!split_pass<Cfg>(e, blk, g, again != 0, left)) return;
    extern __shared__ __align__(16) unsigned char smem[];
    const int* const s_left = reinterpret_cast<const int*>(smem + Cfg::LEFT);
    float* const sm = reinterpret_cast<float*>(smem);
    unsigned* const s_vm = reinterpret_cast<unsigned*>(sm + kF32Smem);
    const int th = g.p0, tw = g.p1, mt = by_reciprocal((int)blk, g.per_NT), n0 = ((int)blk - mt * g.NT) * 32;
    const int ty = by_reciprocal(mt, g.per_tiles_x), wy0 = ty * th, wx0 = (mt - ty * g.tiles_x) * tw;
    const int nty = wy0 + th < e.Hp ? th : e.Hp - wy0, ntx = wx0 + tw < e.Wp ? tw : e.Wp - wx0;
    for (int r = 0; r < nty; ++r)
        for (int x = wx0 & ~15; x < wx0 + ntx; x += 16) {
            const int lx = x - wx0 + (int)threadIdx.x;
            if (!__syncthreads_or(threadIdx.x < 16 && (unsigned)lx < (unsigned)ntx && s_left[r * tw + lx])) continue;
            f32_tile(e, wy0 + r, x, 1, 16, n0, true, sm, s_vm, s_vm + kF32Px, [&](int, int wx, int c) -> unsigned {
                return (unsigned)(wx - wx0) < (unsigned)ntx ? (unsigned)s_left[r * tw + wx - wx0] >> c & 0xffu : 0u;
            });
        }
}

}  // namespace mdcnn
