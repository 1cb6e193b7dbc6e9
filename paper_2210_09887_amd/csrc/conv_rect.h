// Convolution tile of the 3 x 3 fp16 layers of 64 n input channels, and of those of 32 n with stride 2.
#pragma once

#include <type_traits>

#include "conv_device.h"

namespace mdcnn {

// ---------------------------------------------------------------------------
// A tile is a th x tw rectangle of the padded window (tw <= 14, stride 2: 7;
// th * tw <= M) x BN couts, weights in the packed order [tap][cin/16][cout][16]
// (k_pack_weights).  The source pixels it reads, (th + 2) x (tw + 2) of them
// (stride 2: (2 th + 1) x (2 tw + 1)) in rows of 16, are staged per 64-channel
// chunk, 128 bytes a pixel (32 channels, 64 bytes where 64 do not divide): global memory -> LDS without a
// register in between (buffer loads with the lds flag: a wave places 1 KiB at a
// time, 8 pixels).  A pixel out of view or not updated is loaded from beyond the
// end of the delta map, which places zeros, and that is all the masking the taps
// need.  Rows of 128 bytes would put the same piece of every other pixel on the
// same banks, and these loads cannot pad a row, so piece p of pixel x sits at
// p ^ (x % 8): the lane that fetches a piece asks for the one that belongs
// there.  Eight neighbouring pixels are apart, sixteen are not (pixels x and x + 8
// share their banks), nor are the rows of a tile: 4.9 to 6.7 conflict cycles per
// LDS instruction are left.  With rows of 16 pixels the place of a tap's piece is
// one of three registers (dx) plus a constant (dy).
//
// The four waves are WMV (groups of row tiles) x WK (16-channel blocks of a
// chunk); a wave multiplies its row tiles x TN 32 x 32 accumulators over its
// blocks of every tap and loads exactly the weight fragments it needs, RING - 1
// steps ahead.  Two chunks are staged ahead; the loads of the next but one go
// out when a chunk begins, behind the weights of the first steps, so that a
// chunk boundary is one barrier.  The partial sums of the K split are added
// through LDS in the order of the waves, PT row tiles of a wave at a time.
// Chunks, taps and blocks of an entry are walked in the same order whatever the
// tile, so tiles of one WK give the same bits.
//
// What bounds it: the matrix instruction where the channels are many (512 -> 512 on a 66 x 66 window, dense: 12.9 us of K loop in
// a 20 us tile, 93 % of what a loop of nothing else reaches), instruction latency and round trips around the loop where they
// are few: descriptor and flags 0.9 us, rows 0.6, ranks 0.35, sums and pending update 1.0 for 96 entries.  Before, with rows
// staged through registers a chunk at a time and the K loop at 49 % of the pipe: ResNet-18-style 512 x 512 frame 425 -> 387
// us, 30 frames 7.11 -> 6.91 ms, 16 videos 13.4 -> 13.0 ms, HRNet-like 384 x 288 frame 565 -> 520 us (rect_choice: by layer).
// ---------------------------------------------------------------------------
typedef int i32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ i32x4_t raw_rsrc(const void* p, unsigned bytes) {
    const unsigned long long a = (unsigned long long)(uintptr_t)p;
    return i32x4_t{(int)(unsigned)a, (int)(unsigned)(a >> 32), (int)bytes, 0x00020000};
}
// 16 bytes per lane to LDS bytes [lds, lds + 1024), lane after lane.  Written as assembly so that the compiler does not take
// the LDS reads that follow for readers of these bytes: who reads them waits with dma_wait and a barrier.
__device__ __forceinline__ void dma16(i32x4_t rs, unsigned lds, unsigned lane_bytes, unsigned wave_bytes) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds), "v"(lane_bytes), "s"(rs), "s"(wave_bytes) : "memory", "m0");
}
template <int LEFT>
__device__ __forceinline__ void dma_wait() {               // until all but the last LEFT loads of the wave are done
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LEFT) : "memory");
}

// Order of a step with L LDS reads and TN global loads for later steps and L * TN matrix instructions: the loads spread between them.
template <int L, int TN, int Q = 0>
__device__ __forceinline__ void spread() {
    if constexpr (Q < (L > TN ? L : TN)) {
        if constexpr (Q < L) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        if constexpr (Q < TN) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, L > TN ? TN : L, 0);
        spread<L, TN, Q + 1>();
    }
}

// S: stride of the convolution; KB: 16-channel blocks of a chunk (4, or 2 where the channels are no multiple of 64).
template <int WMV_, int WK_, int TM_, int TN_, int NLD_, int RING_, int PT_, int MINB_, int NBUF_ = 2, int S_ = 1, int KB_ = 4>
struct RectCfg {
    static constexpr int WMV = WMV_, WK = WK_, TM = TM_, TN = TN_, NLD = NLD_, RING = RING_, PT = PT_, MINB = MINB_, NBUF = NBUF_, S = S_, KB = KB_;
    static constexpr int M = 32 * WMV * TM, BN = 32 * TN;
    static constexpr int MB = KB / WK;               // 16-channel blocks of a chunk per wave
    static constexpr int NS = 9 * MB;                // steps per chunk and wave
    static constexpr int PXB = 32 * KB;              // bytes of a staged pixel
    static constexpr int ROWB = 16 * PXB;            //       of a staged row of 16 pixels
    static constexpr int LPP = PXB / 16;             // pieces of a pixel, a lane each
    static constexpr int WPR = ROWB / 1024;          // waves that stage a row together
    static constexpr int RPJ = 4 / WPR;              // rows the four waves stage at a time
    static constexpr int ROWS = RPJ * NLD;
    static constexpr int BUF = ROWS * ROWB;          // bytes of a staged chunk
    static constexpr int LDC = BN + 4;               // partial-sum row, floats
    static constexpr int CROWS = 32 * WMV * PT;      // entries per pass of the epilogue
    static constexpr int SUM_BYTES = WK * CROWS * LDC * 4;
    static constexpr int MAIN_BYTES = NBUF * BUF > SUM_BYTES ? NBUF * BUF : SUM_BYTES;
    static constexpr int SMEM = MAIN_BYTES + M * 4 + 64 * 2;
    static_assert(WMV * WK == 4 && KB % WK == 0 && (2 * NS) % RING == 0 && 2 * NS > RING, "four waves; static ring slots over a pair of chunks");
    static_assert((RING - 1) * TN + NLD < 63, "the counter of outstanding loads has six bits");
};

// The tiles in use, by their entries.  All but the last split the channels four ways and give the same bits.
template <int TN>
struct RectTiles {
    using T64 = RectCfg<1, 4, 2, TN, 5, 9, 2, 2>;
    using T96 = RectCfg<1, 4, 3, TN, 5, 6, 2, 2>;
    using T128 = RectCfg<1, 4, 4, TN, 6, TN == 1 ? 6 : 3, 2, 2>;
    using T160 = RectCfg<1, 4, 5, TN, 7, 9, 3, 1>;
    using T256 = RectCfg<4, 1, 2, TN, 10, 6, 2, 2, 1>;       // 64 input channels only
    // stride 2, 64 entries: 64 input channels, 64 n, 32 n
    using S2One = RectCfg<1, 4, 2, TN, 10, TN == 4 ? 3 : 9, 1, 2, 1, 2>;
    using S2 = RectCfg<1, 4, 2, TN, 8, TN == 4 ? 3 : 9, 1, 2, 2, 2>;
    using S2Half = RectCfg<2, 2, 1, TN, 5, 9, 1, 2, 2, 2, 2>;
};

template <typename Cfg>
constexpr int rect_body_number() {
    return Cfg::S == 1 ? multi_rect_body(Cfg::M, Cfg::TN) : multi_rect_body(Cfg::KB == 2 ? kRectS2Half : Cfg::NBUF == 1 ? kRectS2One : kRectS2, Cfg::TN);
}

// blk: the tile.  READ: the launch may read the destination out (EdgeDev::dY).
template <typename Cfg, bool READ>
__device__ __forceinline__ void rect_body(const EdgeDev& e, unsigned blk, const TileGrid& g) {
    constexpr int WMV = Cfg::WMV, WK = Cfg::WK, TM = Cfg::TM, TN = Cfg::TN, NLD = Cfg::NLD, MB = Cfg::MB, NS = Cfg::NS, D = Cfg::RING,
                  M = Cfg::M, BN = Cfg::BN, LDC = Cfg::LDC, PT = Cfg::PT, S = Cfg::S, PXB = Cfg::PXB, ROWB = Cfg::ROWB, LPP = Cfg::LPP, WPR = Cfg::WPR, RPJ = Cfg::RPJ;
    extern __shared__ __align__(16) unsigned char smem[];
    float* const sC = reinterpret_cast<float*>(smem);
    int* const s_ent = reinterpret_cast<int*>(smem + Cfg::MAIN_BYTES);      // entry -> ly << 4 | lx
    unsigned char* const s_mask = smem + Cfg::MAIN_BYTES + M * 4;           // live pixels of a staged row, 16 bits each
    // (fetched field by field where they are used: 1 us until the flags are asked for)
    int Hp = e.Hp, Wp = e.Wp, sH = e.sH, sW = e.sW, Cin = e.Cin, Cout = e.Cout, by0 = e.by0, bx0 = e.bx0, pad = e.pad, p_oy = e.p_oy, p_ox = e.p_ox;
    const void *delta = e.delta, *wp = e.wp;
    const uint8_t* sflags = e.sflags;
    f16 *P = (f16*)e.P, *out_p = (f16*)e.dY;
    int dH = e.dH, dW = e.dW, relu = e.s_relu;
    int NT = g.NT, th = g.p0, tw = g.p1, tiles_x = g.tiles_x;
    unsigned per_NT = g.per_NT, per_tiles_x = g.per_tiles_x;
    read_now(Hp, Wp, sH, sW, Cin, Cout, by0, bx0, pad, p_oy, p_ox, delta, wp, sflags, P, NT, th, tw, tiles_x, per_NT, per_tiles_x);
    if constexpr (READ) read_now(out_p, dH, dW, relu);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WMV, wk = wave / WMV;
    const int r32 = lane & 31, kh = lane >> 5;
    const int nchunks = Cfg::NBUF > 1 ? Cin / (16 * Cfg::KB) : 1;
    const unsigned row = (unsigned)Cin * 2u;         // bytes of a source pixel
    constexpr unsigned kOutside = 0x80000000u;       // past the end of every tensor
    // (the host checks that both tensors are smaller than 2 GiB)
    const i32x4_t drs = raw_rsrc(delta, (unsigned)sH * (unsigned)sW * row);
    const rsrc_t frs = make_rsrc(sflags, (unsigned)sH * (unsigned)sW);
    const rsrc_t wrs = make_rsrc(wp, 9u * (unsigned)Cin * (unsigned)Cout * 2u);
    const unsigned tap_stride = (unsigned)(Cin / 16) * (unsigned)Cout * 32u;   // packed weights: bytes per tap
    const unsigned blk_stride = (unsigned)Cout * 32u;                          //                 per 16-channel block
    const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem);

    const int mt = by_reciprocal((int)blk, per_NT), nt = (int)blk - mt * NT;   // blk % 8 picks the XCD: few cout tiles per XCD
    const int n0 = nt * BN;
    const unsigned wlane = (unsigned)(r32 * 16 + kh * 8) * 2u;                      // this lane's bytes within a fragment
    const unsigned wwave = ((unsigned)wk * (unsigned)Cout + (unsigned)n0) * 32u;   // this wave's K block and cout tile
    f16x8 fa[D][TN];                                  // weight fragments in flight
    auto load_a = [&](int slot, int c, int i) {       // step i of chunk c; i may run into the next chunk
        const int cc = i < NS ? c : (c + 1 < nchunks ? c + 1 : c), ii = i < NS ? i : i - NS;
        const unsigned src = wwave + (unsigned)(ii / MB) * tap_stride + (unsigned)(cc * Cfg::KB + WK * (ii % MB)) * blk_stride;
#pragma unroll
        for (int j = 0; j < TN; ++j) fa[slot][j] = buf_load16(wrs, wlane, src + (unsigned)j * 32u * 32u);
    };
    const int ty = by_reciprocal(mt, per_tiles_x), tx = mt - ty * tiles_x;
    const int wy0 = ty * th, wx0 = tx * tw;
    const int nty = wy0 + th < Hp ? th : Hp - wy0, ntx = wx0 + tw < Wp ? tw : Wp - wx0;
    // where piece p of pixel x of a row lies: at p ^ swz(x)
    auto swz = [](int x) { return LPP == 8 ? (S == 1 ? x & 7 : x >> 1) : x >> 2; };
    // staged pixels of this thread: rows RPJ j + row0, column sx, 16-byte piece lane % LPP of the pixel in LDS
    const int row0 = wave / WPR, sx = (wave % WPR) * (16 / WPR) + lane / LPP, ix = (wx0 - bx0) * S - pad + sx, iy = (wy0 - by0) * S - pad + row0;
    const int nsy = (nty - 1) * S + 3, nsx = (ntx - 1) * S + 3;              // staged rows, columns
    const unsigned out = sx < nsx && ix >= 0 && ix < sW ? 0u : kOutside;
    const unsigned pix = (unsigned)(iy * sW + ix), piece = (unsigned)((lane % LPP) ^ swz(sx)) * 16u;
    unsigned fl[NLD], hsrc[NLD];
#pragma unroll
    for (int j = 0; j < NLD; ++j) {                   // (a flag outside the source reads as 0)
        const bool in = RPJ * j + row0 < nsy && iy + RPJ * j >= 0 && iy + RPJ * j < sH;
        fl[j] = __builtin_amdgcn_raw_buffer_load_b8(frs, (int)(in ? (pix + (unsigned)(RPJ * j * sW)) | out : kOutside), 0, 0);
    }
    // loads come back in order: the weights of the first steps, the slowest here, behind the flags
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < D - 1; ++i) load_a(i, 0, i);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < NLD; ++j) hsrc[j] = ((pix + (unsigned)(RPJ * j * sW)) * row + piece) | (~fl[j] >> 2) << 31;      // kFlagM == 4
    auto stage = [&](int c) {                          // chunk c -> its buffer
#pragma unroll
        for (int j = 0; j < NLD; ++j)
            dma16(drs, lds0 + (unsigned)((c & 1) * Cfg::BUF + (wave + 4 * j) * 1024), hsrc[j], (unsigned)(c * PXB));
    };
    stage(0);
    if (nchunks > 1) stage(1);
    unsigned short bits[NLD];
#pragma unroll
    for (int j = 0; j < NLD; ++j) {
        if constexpr (LPP == 8) {
            const unsigned long long b = __ballot(fl[j] & kFlagM) & 0x0101010101010101ull;         // eight lanes to a pixel
            bits[j] = (unsigned char)((b * 0x0102040810204080ull) >> 56);
        } else {
            unsigned long long b = __ballot(fl[j] & kFlagM) & 0x1111111111111111ull;               // four
            b = (b | b >> 3) & 0x0303030303030303ull;
            b = (b | b >> 6) & 0x000f000f000f000full;
            b = (b | b >> 12) & 0x000000ff000000ffull;
            bits[j] = (unsigned short)(b | b >> 24);
        }
    }
    if (lane == 0) {
#pragma unroll
        for (int j = 0; j < NLD; ++j) {
            if constexpr (LPP == 8) s_mask[(2 * j + row0) * 2 + (wave & 1)] = (unsigned char)bits[j];
            else reinterpret_cast<unsigned short*>(s_mask)[4 * j + row0] = bits[j];
        }
    }
    __syncthreads();
    // the live pixels of the tile, ranked row by row: lane l of every wave has row l
    int any = 0, upto = 0;
    if (lane < nty) {
        const unsigned short* r = reinterpret_cast<const unsigned short*>(s_mask) + lane * S;
        int m = r[0] | r[1] | r[2];
        m = m | m >> 1 | m >> 2;
        if constexpr (S == 2) {                       // every other column
            m &= 0x5555;
            m = (m | m >> 1) & 0x3333;
            m = (m | m >> 2) & 0x0f0f;
            m = m | m >> 4;
        }
        any = m & ((1 << ntx) - 1);
    }
    upto = __popc(any);
    upto += __builtin_amdgcn_update_dpp(0, upto, 0x111, 0xf, 0xf, false);      // row_shr:1, 2, 4, 8: sums within 16 lanes
    upto += __builtin_amdgcn_update_dpp(0, upto, 0x112, 0xf, 0xf, false);
    upto += __builtin_amdgcn_update_dpp(0, upto, 0x114, 0xf, 0xf, false);
    upto += __builtin_amdgcn_update_dpp(0, upto, 0x118, 0xf, 0xf, false);
    upto += __builtin_amdgcn_update_dpp(0, upto, 0x142, 0xa, 0xf, false);      // row_bcast:15: those of the first 16 to the next
    const int tot = __builtin_amdgcn_readlane(upto, 31);
    if (tot == 0) {
        dma_wait<0>();
        return;
    }
    const float rtw = rcp_of(tw);
#pragma unroll
    for (int t = tid; t < M; t += 256) {
        const int ly = fast_div(t, tw, rtw), lx = t - ly * tw;
        const int a = __shfl(any, ly), before = __shfl(upto, ly) - __popc(a);
        if (ly < nty && (a >> lx & 1)) s_ent[before + __popc(a & ((1 << lx) - 1))] = ly << 4 | lx;
    }
    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    if (nchunks > 1) dma_wait<NLD>();
    else dma_wait<0>();
    __syncthreads();

    const int nrt = (tot + 31) >> 5;                  // live 32-entry row tiles of the tile
    const int mylive = nrt > wm ? (nrt - wm + WMV - 1) / WMV : 0;      // of this wave: row tiles wm, wm + WMV, ...
    int off[TM][3];                                   // bytes of this lane's piece at taps (0, dx)
#pragma unroll
    for (int t = 0; t < TM; ++t) {
        const int r = (t * WMV + wm) * 32 + r32, ent = s_ent[r < tot ? r : 0];
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) {
            const int x = (ent & 15) * S + dx;
            off[t][dx] = ((ent >> 4) * S * 16 + x) * PXB + (((2 * wk + kh) ^ swz(x)) << 4);
        }
    }

    // The K loop for L live row tiles of this wave.  Step i of a chunk: tap i / MB, 16-channel block wk + WK * (i % MB).
    auto kloop = [&](auto lc) {
        constexpr int L = decltype(lc)::value;
        f16x8 fb[2][L > 0 ? L : 1];
        auto chunk = [&](auto par, int c) {
            constexpr int P = decltype(par)::value;
            auto load_b = [&](int slot, int i) {
                const int tap = i / MB, flip = (WK * (i % MB)) * 2 * 16;         // block wk + WK q: another bit of the piece number
#pragma unroll
                for (int t = 0; t < L; ++t)
                    fb[slot][t] = *reinterpret_cast<const f16x8*>(smem + P * Cfg::BUF + (tap / 3) * ROWB + (off[t][tap % 3] ^ flip));
            };
            if (c > 0 && c + 1 < nchunks) stage(c + 1);
            load_b(0, 0);
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                const int g = P * NS + i;                            // ring slots run on over a pair of chunks
                load_a((g + D - 1) % D, c, i + D - 1);
                if (i + 1 < NS) load_b((i + 1) & 1, i + 1);
#pragma unroll
                for (int t = 0; t < L; ++t)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[t][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[g % D][j], fb[i & 1][t], acc[t][j], 0, 0, 0);
                // the loads just issued (for later steps) stay ahead of these MFMAs and are spread between them
                spread<L, TN>();
                __builtin_amdgcn_sched_barrier(0);
            }
            if (c + 1 < nchunks) {
                dma_wait<(D - 1) * TN>();             // the next chunk is older than the weights in flight
                __syncthreads();
            }
        };
        for (int c = 0; c < nchunks; c += 2) {
            chunk(std::integral_constant<int, 0>{}, c);
            if (c + 1 < nchunks) chunk(std::integral_constant<int, 1>{}, c + 1);
        }
    };
    switch (mylive) {
        case 0: kloop(std::integral_constant<int, 0>{}); break;
        case 1: kloop(std::integral_constant<int, 1>{}); break;
        case 2: kloop(std::integral_constant<int, TM >= 2 ? 2 : TM>{}); break;
        case 3: kloop(std::integral_constant<int, TM >= 3 ? 3 : TM>{}); break;
        case 4: kloop(std::integral_constant<int, TM >= 4 ? 4 : TM>{}); break;
        default: kloop(std::integral_constant<int, TM>{}); break;
    }

    // P <- P + sum, PT row tiles of every wave at a time
    constexpr int TPR = BN / 8;                        // threads per entry, 8 couts each
    constexpr int RPP = 256 / TPR, NPASS = (Cfg::CROWS + RPP - 1) / RPP;
    const int c8 = (tid % TPR) * 8;
#pragma unroll
    for (int q = 0; q < TM; q += PT) {
        if (q * WMV >= nrt) break;                    // block-uniform
        f16x8 pold[NPASS];
        f16* pp[NPASS];
#pragma unroll
        for (int t = 0; t < NPASS; ++t) {              // all reads go out together; dead rows read entry 0 and store nothing
            const int srow = tid / TPR + t * RPP, at = q * WMV * 32 + srow, en = s_ent[srow < Cfg::CROWS && at < tot ? at : 0];
            pp[t] = P + ((size_t)wrapc(p_oy + wy0 + (en >> 4), Hp) * Wp + wrapc(p_ox + wx0 + (en & 15), Wp)) * Cout + n0 + c8;
            pold[t] = *reinterpret_cast<const f16x8*>(pp[t]);
        }
        __syncthreads();                              // the staged rows, or the sums of the last pass, have been read
#pragma unroll
        for (int i = q; i < q + PT && i < TM; ++i) {
            if (i >= mylive) continue;
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                float* dst = sC + (wk * Cfg::CROWS + ((i - q) * WMV + wm) * 32 + r32) * LDC + j * 32 + 4 * kh;
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    *reinterpret_cast<float4*>(dst + 8 * g) = make_float4(acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
            }
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < NPASS; ++t) {
            const int srow = tid / TPR + t * RPP, at = q * WMV * 32 + srow;
            if (srow < Cfg::CROWS && at < tot) {
                float v[8];
#pragma unroll
                for (int kq = 0; kq < WK; ++kq) {
                    const float* src = sC + (kq * Cfg::CROWS + srow) * LDC + c8;
                    const float4 v0 = *reinterpret_cast<const float4*>(src), v1 = *reinterpret_cast<const float4*>(src + 4);
                    const float part[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
#pragma unroll
                    for (int c = 0; c < 8; ++c) v[c] = kq ? v[c] + part[c] : part[c];
                }
                f16x8 o = pold[t];
#pragma unroll
                for (int c = 0; c < 8; ++c) o[c] = (f16)((float)o[c] + v[c]);
                *reinterpret_cast<f16x8*>(pp[t]) = o;
                if (READ && out_p) {                  // (the launch reads the site out)
                    const int en = s_ent[at], oy = wy0 + (en >> 4) - by0, ox = wx0 + (en & 15) - bx0;
                    if ((unsigned)oy < (unsigned)dH && (unsigned)ox < (unsigned)dW)
                        write_out<f16, 8>(out_p, relu, ((size_t)oy * dW + ox) * Cout + n0 + c8, reinterpret_cast<const f16*>(&o));
                }
            }
        }
    }
}

}  // namespace mdcnn
