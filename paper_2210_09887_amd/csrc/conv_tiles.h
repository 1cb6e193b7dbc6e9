// Convolution tiles on the matrix cores (fp16): the gather-GEMM tile and the halo-staged tile, as device functions that
// a kernel of one edge (kernels_conv.hip) or of several independent edges (kernels_multi.hip) runs.
#pragma once

#include <type_traits>

#include "conv_device.h"

namespace mdcnn {

// ---------------------------------------------------------------------------
// Tiled MFMA gather-GEMM (the fast path for fp16 layers with Cin % 32 == 0).
// Block tile = BM list entries (pixels) x BN couts, 4 waves arranged WM x WN,
// each wave owning TM x TN 32x32 accumulators.  K runs over (active tap,
// KC-channel chunk) steps; per step the weight slab [BN][KC] and the gathered
// delta slab [BM][KC] (rows of taps that miss the update mask are zero) go
// global -> registers -> LDS (rows padded by 16 bytes) while the previous step is
// multiplied out of LDS.  Taps no entry of the tile uses are skipped.  The
// accumulators are transposed through LDS so that P is updated with 16-byte
// accesses that are contiguous along the channels.
// v_mfma_f32_32x32x16_f16: operand A = 32 couts x 16 cin (weights), operand
// B = 16 cin x 32 pixels; lane l feeds row/col l%32 with the 8 consecutive cin
// starting at 8*(l/32); the result puts pixel l%32 on lane l with couts
// 8*(r/4) + 4*(l/32) + r%4 in accumulator register r.
// ---------------------------------------------------------------------------
template <int WM, int WN, int TM, int TN, int KC, int PIPE>
struct TiledCfg {
    static constexpr int BM = 32 * WM * TM, BN = 32 * WN * TN;
    static constexpr int LDK = KC + 8;             // slab row, halves
    static constexpr int LDC = BN + 4;             // transposed accumulator row, floats
    static constexpr int CPR = KC / 8;             // 16-byte chunks per slab row
    static constexpr int STAGE_HALVES = (BM + BN) * LDK;
    static constexpr int SLAB_BYTES = PIPE * STAGE_HALVES * 2;
    static constexpr int C_BYTES = BM * LDC * 4;
    static constexpr int MAIN_BYTES = SLAB_BYTES > C_BYTES ? SLAB_BYTES : C_BYTES;
    static constexpr int SMEM = MAIN_BYTES + (4 * BM + 8) * 4;      // + the entries' rows and a few counts
    static constexpr int TPS = kSegPixels / BM;    // tiles per list segment
    // Blocks a compute unit is to hold: what fits its LDS, as far as the accumulators leave registers.  The kernel is bounded by
    // the round trips of its gathers, which the other blocks cover.  Left to itself the compiler takes a few registers more than
    // a wave's share: 16 videos, 128 -> 256 channels, stride 2 on 128 x 128 (64 x 64 tiles of 128 channels, 130 registers, three
    // blocks) 99.3 us, with four 89.9; 64 -> 128 on 256 x 256 111 and 100 us, its 1x1 50 and 43.
    static constexpr int FIT = 160 * 1024 / SMEM, ROOM = TM * TN == 1 ? 4 : TM * TN == 2 ? 3 : TM * TN == 4 ? 2 : 1;
    static constexpr int WAVES = PIPE > 1 || FIT < 1 ? 1 : FIT < ROOM ? FIT : ROOM;
};

// Work item u of a 1-D grid -> (pixel tile m, cout tile n).  Work groups are
// dealt round-robin to the 8 XCDs, each with its own L2: tying u % 8 to the
// cout tile makes all blocks of one XCD share the same weight slice.
__device__ __forceinline__ void map_tile(int u, int NT, int xcd_map, int& m, int& n) {
    if (xcd_map) {
        const int q = 8 / NT, x = u & 7, r = u >> 3;
        n = x % NT;
        m = r * q + x / NT;
    } else {
        n = u % NT;
        m = u / NT;
    }
}

// PIPE = 1: one LDS buffer, loads one step ahead (two barriers per step).
// PIPE = 2: two LDS buffers and two register stages, loads two steps ahead
//           (one barrier per step).
// blk, nblk: this block's number among the blocks that work on tiles of the edge.  Others make the by-products (1x1 and 3x3
// layers; for others every tile makes them itself).  READ: the launch may read the destination out (EdgeDev::dY).
template <int WM, int WN, int TM, int TN, int KC, int PIPE, bool READ>
__device__ __forceinline__ void tiled_body(const EdgeDev& e, unsigned blk, unsigned nblk, TileGrid g, int work_items) {
    int NT = g.NT, xcd_map = g.p0;
    // (the descriptor's fields are fetched where they are used: all held from the start, bottleneck 44.0 against 43.6 us, HRNet-like
    // frame 478 against 473)
    read_now(NT, xcd_map, work_items);
    const bool published = e.k == 1 || e.k == 3;
    using Cfg = TiledCfg<WM, WN, TM, TN, KC, PIPE>;
    constexpr int BM = Cfg::BM, BN = Cfg::BN, LDK = Cfg::LDK, LDC = Cfg::LDC, CPR = Cfg::CPR, TPS = Cfg::TPS;
    constexpr int NB = (BM * CPR + 255) / 256, NA = (BN * CPR + 255) / 256;
    static_assert(WM * WN == 4 && kSegPixels % BM == 0, "4 waves; tiles do not straddle segments");
    extern __shared__ __align__(16) unsigned char smem[];
    f16* slab = reinterpret_cast<f16*>(smem);            // PIPE x { [BM][LDK] deltas, [BN][LDK] weights }
    float* sC = reinterpret_cast<float*>(smem);          // [BM][LDC] after the K loop
    int* const s_base = reinterpret_cast<int*>(smem + Cfg::MAIN_BYTES);
    int *const s_wy = s_base + BM, *const s_wx = s_wy + BM, *const sh = s_wx + BM;
    unsigned* const s_vm = reinterpret_cast<unsigned*>(sh + 8);

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave % WM, wn = wave / WM;
    const int r32 = lane & 31, kh = lane >> 5;
    const int MT = edge_segments(e) * TPS;
    // (the host checks that both tensors are smaller than 2 GiB)
    const rsrc_t drs = make_rsrc(e.delta, (unsigned)e.sH * (unsigned)e.sW * (unsigned)e.Cin * 2u);
    const rsrc_t wrs = make_rsrc(e.w, (unsigned)(e.k * e.k) * (unsigned)e.Cin * (unsigned)e.Cout * 2u);

    if (!published) carry_source_compaction(e, sh, blk, nblk);

    // The f x f pixels an entry of an upsampling edge adds to are dealt to f * f / 4 items, which all make the entry's sums
    // (a 1x1 convolution: a step or two): in one block they were up to 64 read-add-write round trips in a row (12 x 9 source
    // pixels, 256 -> 32 channels, 8-fold: 31 us, now 12).
    const int f = 1 << e.up, splits = f > 2 ? f * f / 4 : 1, split_items = work_items / splits;
    for (int u = (int)blk; u < work_items; u += (int)nblk) {
        const int part = u / split_items;                 // (0 without upsampling)
        int mt, nt;
        map_tile(u - part * split_items, NT, xcd_map, mt, nt);
        if (mt >= MT) continue;
        const int seg = mt / TPS, first = (mt - seg * TPS) * BM;
        const int n0 = nt * BN;
        __syncthreads();                                  // previous tile is done with LDS
        const int tot = tile_prologue(e, seg, first, BM, nt == 0 && first == 0 && !e.up && !published, nt == 0 && !e.up && !published,
                                      s_base, s_wy, s_wx, s_vm, sh);
        const int live = tot - first < BM ? tot - first : BM;     // entries of this tile (block-uniform)
        if (live <= 0) continue;
        const unsigned tilemask = (unsigned)sh[5];
        if (tid == 0 && nt == 0 && part == 0 && (e.up || !published)) add_macs(e, sh[4], 0);    // statistics: one atomic per tile

        f32x16 acc[TM][TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

        // Per-thread chunk descriptors of this tile: which slab rows this thread
        // moves, their source offsets (elements) and tap masks.  Per step only a
        // block-uniform offset is added; a row whose tap misses the update mask is
        // loaded from beyond the end of the tensor, which a buffer load answers with
        // zeros (no divergent branches and no selects on the data in the K loop).
        int offB[NB];
        unsigned offA[NA];
        unsigned vmB[NB];
        int ldsB[NB], ldsA[NA];
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int ch = tid + 256 * i;
            const int row = (ch / CPR) % BM, cc = ch % CPR;          // % BM: keep partial last rounds in range
            offB[i] = (s_base[row] * e.Cin + cc * 8) * 2;      // bytes; may be negative: the top left tap of a border pixel
            vmB[i] = (BM * CPR) % 256 == 0 || ch < BM * CPR ? s_vm[row] : 0u;
            ldsB[i] = row * LDK + cc * 8;
        }
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int ch = tid + 256 * i;
            const int row = (ch / CPR) % BN, cc = ch % CPR;
            offA[i] = ((unsigned)(n0 + row) * (unsigned)e.Cin + cc * 8) * 2u;      // bytes
            ldsA[i] = row * LDK + cc * 8;
        }
        const unsigned tap_stride_w = (unsigned)e.Cout * (unsigned)e.Cin * 2u;    // bytes

        // the load iterator runs PIPE steps ahead of the multiplication
        unsigned ld_rem = tilemask;
        int ld_tap = ld_rem ? __ffs(ld_rem) - 1 : -1, ld_c0 = 0;
        f16x8 rb[PIPE][NB], ra[PIPE][NA];
        auto load_next = [&](auto stage) {
            constexpr int S = decltype(stage)::value;
            if (ld_tap < 0) return;
            const int jy = ld_tap / e.k, jx = ld_tap - jy * e.k;
            const int stepB = ((jy * e.sW + jx) * e.Cin + ld_c0) * 2;                 // block-uniform, bytes
            const unsigned stepA = (unsigned)ld_tap * tap_stride_w + (unsigned)ld_c0 * 2u;
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const bool valid = (vmB[i] >> ld_tap) & 1u;                           // then offB + stepB is a pixel of the source
                rb[S][i] = buf_load16(drs, valid ? (unsigned)(offB[i] + stepB) : 0x80000000u, 0u);
            }
#pragma unroll
            for (int i = 0; i < NA; ++i) ra[S][i] = buf_load16(wrs, offA[i], stepA);
            ld_c0 += KC;
            if (ld_c0 >= e.Cin) { ld_c0 = 0; ld_rem &= ld_rem - 1; ld_tap = ld_rem ? __ffs(ld_rem) - 1 : -1; }
        };
        auto store_stage = [&](auto stage) {
            constexpr int S = decltype(stage)::value;
            f16* sB = slab + S * Cfg::STAGE_HALVES;
            f16* sA = sB + BM * LDK;
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                if ((BM * CPR) % 256 == 0 || tid + 256 * i < BM * CPR) *reinterpret_cast<f16x8*>(sB + ldsB[i]) = rb[S][i];
            }
#pragma unroll
            for (int i = 0; i < NA; ++i)
                if ((BN * CPR) % 256 == 0 || tid + 256 * i < BN * CPR) *reinterpret_cast<f16x8*>(sA + ldsA[i]) = ra[S][i];
        };
        auto multiply = [&](auto stage) {
            constexpr int S = decltype(stage)::value;
            constexpr int KK = KC / 16;
            const f16* sB = slab + S * Cfg::STAGE_HALVES + (wm * TM * 32 + r32) * LDK + kh * 8;
            const f16* sA = slab + S * Cfg::STAGE_HALVES + BM * LDK + (wn * TN * 32 + r32) * LDK + kh * 8;
            f16x8 fb[KK][TM], fa[KK][TN];                    // all fragments of the step, then the MFMAs
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
#pragma unroll
                for (int i = 0; i < TM; ++i) fb[kk][i] = *reinterpret_cast<const f16x8*>(sB + i * 32 * LDK + kk * 16);
#pragma unroll
                for (int j = 0; j < TN; ++j) fa[kk][j] = *reinterpret_cast<const f16x8*>(sA + j * 32 * LDK + kk * 16);
            }
#pragma unroll
            for (int kk = 0; kk < KK; ++kk)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[kk][j], fb[kk][i], acc[i][j], 0, 0, 0);
        };
        using S0 = std::integral_constant<int, 0>;
        using S1 = std::integral_constant<int, PIPE - 1>;
        int steps = __popc(tilemask) * (e.Cin / KC);
        if constexpr (PIPE == 1) {
            load_next(S0{});
            store_stage(S0{});
            __syncthreads();
            while (steps > 0) {
                load_next(S0{});                             // in flight while this step is multiplied
                multiply(S0{});
                __syncthreads();
                if (--steps > 0) store_stage(S0{});
                __syncthreads();
            }
        } else {
            load_next(S0{});
            load_next(S1{});
            while (steps > 0) {
                store_stage(S0{});
                load_next(S0{});                             // refill the registers just drained
                __syncthreads();
                multiply(S0{});
                if (--steps == 0) break;
                store_stage(S1{});
                load_next(S1{});
                __syncthreads();
                multiply(S1{});
                --steps;
            }
            __syncthreads();                                 // all multiplications done: LDS becomes the C tile
        }

        // accumulators -> LDS as [pixel][cout]
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                float* dst = sC + ((wm * TM + i) * 32 + r32) * LDC + (wn * TN + j) * 32 + 4 * kh;
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    *reinterpret_cast<float4*>(dst + 8 * g) =
                        make_float4(acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
            }
        __syncthreads();
        constexpr int TPR = BN / 8;                        // threads per pixel row, 8 couts each
        const int c8 = (tid % TPR) * 8;
        if (f == 1) {
            // P <- P + sum: all reads of P go out first (their latency is paid once), then the stores
            constexpr int RPP = 256 / TPR, NPASS = (BM + RPP - 1) / RPP;
            f16x8 pold[NPASS];
            f16* pp[NPASS];
#pragma unroll
            for (int t = 0; t < NPASS; ++t) {
                const int row = tid / TPR + t * RPP;
                const int rr = row < live ? row : 0;        // dead rows read entry 0 and store nothing
                pp[t] = (f16*)e.P + pdst_offset(e, s_wy[rr], s_wx[rr]) + n0 + c8;
                pold[t] = *reinterpret_cast<const f16x8*>(pp[t]);
            }
#pragma unroll
            for (int t = 0; t < NPASS; ++t) {
                const int row = tid / TPR + t * RPP;
                if (row < live) {
                    const float4 v0 = *reinterpret_cast<const float4*>(sC + row * LDC + c8);
                    const float4 v1 = *reinterpret_cast<const float4*>(sC + row * LDC + c8 + 4);
                    const float v[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
                    f16x8 o = pold[t];
#pragma unroll
                    for (int q = 0; q < 8; ++q) o[q] = (f16)((float)o[q] + v[q]);
                    *reinterpret_cast<f16x8*>(pp[t]) = o;
                    if (READ && e.dY) {                     // (the launch reads the site out)
                        const int oy = s_wy[row] - e.by0, ox = s_wx[row] - e.bx0;
                        if ((unsigned)oy < (unsigned)e.dH && (unsigned)ox < (unsigned)e.dW)
                            write_out<f16, 8>((f16*)e.dY, e.s_relu, ((size_t)oy * e.dW + ox) * e.Cout + n0 + c8, reinterpret_cast<const f16*>(&o));
                    }
                }
            }
            continue;
        }
        for (int row = tid / TPR; row < BM && row < live; row += 256 / TPR) {
            const float4 v0 = *reinterpret_cast<const float4*>(sC + row * LDC + c8);
            const float4 v1 = *reinterpret_cast<const float4*>(sC + row * LDC + c8 + 4);
            const float v[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
            f16x8 o[4];
            f16* p[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int at = part * 4 + q;                 // 2-fold: all four
                p[q] = (f16*)e.P + pdst_offset(e, s_wy[row] + (at >> e.up), s_wx[row] + (at & (f - 1))) + n0 + c8;
                o[q] = *reinterpret_cast<f16x8*>(p[q]);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
#pragma unroll
                for (int c = 0; c < 8; ++c) o[q][c] = (f16)((float)o[q][c] + v[c]);
                *reinterpret_cast<f16x8*>(p[q]) = o[q];
                if (nt == 0 && c8 == 0) mark_pixel(e, s_wy[row] + ((part * 4 + q) >> e.up), s_wx[row] + ((part * 4 + q) & (f - 1)));
            }
        }
    }
}

// Variant of tile_prologue for tiles that are index sub-ranges of a segment: the
// tile takes the entries among indices [sub_lo, sub_lo + sub_n) of segment `seg`
// (sub_lo a multiple of 64).  Returns their number; rows s_* are filled for them.
__device__ __forceinline__ int tile_prologue_sub(const EdgeDev& e, int seg, int sub_lo, int sub_n, bool publish, bool touch,
                                                 int* s_wy, int* s_wx, int* sh) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = e.Hp * e.Wp;
    const int p = seg * kSegPixels + tid;
    if (tid == 0) sh[4] = 0;
    int cy = 0, cx = 0, wy = 0, wx = 0;
    unsigned vm = 0;
    if (p < n && tid < kSegPixels) {                       // waves beyond the fourth only keep the barriers
        decode_entry(e, p, cy, cx, wy, wx);
        vm = tap_mask(e, cy, cx);
    }
    const bool has = vm != 0;
    const unsigned long long bal = __ballot(has);
    const int rank = __popcll(bal & ((1ull << lane) - 1ull));
    if (lane == 0 && wave < 4) sh[wave] = __popcll(bal);
    __syncthreads();
    int off = rank, base = 0, cnt = 0;
    for (int i = 0; i < 4; ++i) {
        if (i < wave) off += sh[i];
        if (i * 64 < sub_lo) base += sh[i];
        else if (i * 64 < sub_lo + sub_n) cnt += sh[i];
    }
    const bool mine = has && tid >= sub_lo && tid < sub_lo + sub_n;
    if (mine) {
        s_wy[off - base] = wy;
        s_wx[off - base] = wx;
        if (touch) mark_touched(e, wy, wx);
    }
    if (publish && has) e.clist[seg * kSegPixels + off] = p;
    if (publish && tid == 0) {                             // single writer per segment: no atomics
        const int tot = sh[0] + sh[1] + sh[2] + sh[3];
        e.ccnt[seg] = tot;
        e.cacc[seg] += (unsigned long long)tot;
    }
    const int taps = wave_sum(mine ? __popc(vm) : 0);
    if (lane == 0 && taps) atomicAdd(&sh[4], taps);
    __syncthreads();
    return cnt;
}

// Variant of tile_prologue for tiles that are th x tw rectangles of the padded window (th * tw <= 256, top-left
// corner (wy0, wx0)): thread t looks at tile pixel (t / tw, t % tw); the live ones are ranked in that order.
// Returns their number; rows s_wy / s_wx are filled for them.
// The tap mask of a tile pixel is read off the tile's staged rectangle: s_pix[ry * rw + rx] >= 0 where the source pixel
// (ry, rx) of the rectangle (the tile plus its halo) is in view and updated (3x3, stride 1: the footprint of tile pixel
// (ly, lx) is rectangle rows ly .. ly + 2, columns lx .. lx + 2) - no flag loads of its own.  Nothing is written to global
// memory: what a tile leaves behind besides its sums is done by other blocks (publish_edge).
__device__ __forceinline__ int tile_prologue_2d(const EdgeDev& e, int wy0, int wx0, int th, int tw, const int* s_pix, int rw,
                                                int* s_wy, int* s_wx, int* sh) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ly = fast_div(tid, tw, rcp_of(tw)), lx = tid - ly * tw;
    const int wy = wy0 + ly, wx = wx0 + lx;
    bool has = false;
    if (ly < th && wy < e.Hp && wx < e.Wp) {
        const int* r = s_pix + ly * rw + lx;
        int any = -1;                                      // negative as long as no tap is live
#pragma unroll
        for (int t = 0; t < 9; ++t) any &= r[(t / 3) * rw + t % 3] | 0x7fffffff;
        has = any >= 0;
    }
    const unsigned long long bal = __ballot(has);
    if (lane == 0) sh[wave] = __popcll(bal);
    __syncthreads();
    int off = __popcll(bal & ((1ull << lane) - 1ull));
    for (int i = 0; i < wave; ++i) off += sh[i];
    if (has) {
        s_wy[off] = wy;
        s_wx[off] = wx;
    }
    const int cnt = sh[0] + sh[1] + sh[2] + sh[3];
    __syncthreads();
    return cnt;
}

// ---------------------------------------------------------------------------
// Halo-staged MFMA convolution: KS x KS, stride 1, fp16, weights in the packed
// order [tap][cin/16][cout][16] (k_pack_weights).
// A tile is one NSUB-th of a list segment -- the entries among SUB = kSegPixels
// / NSUB consecutive indices of the padded window -- x BN couts.  Every input
// pixel those entries read lies in a small rectangle of the source (the rows
// the index range spans plus KS-1, full width if it spans more than one row).
// Per KC-channel chunk that rectangle is staged ONCE in LDS -- zero rows for
// pixels out of view or not updated, which is all the masking the taps need --
// and all KS*KS taps multiply out of it: the deltas are fetched once instead
// of once per tap.  The weights never touch LDS: the four waves are WMV
// (row-tile groups) x WK (K split); a wave multiplies its row tiles x TN 32x32
// accumulators over every WK-th 16-channel block of every tap and loads
// exactly the fragments it needs, 1 KiB contiguous each, several steps ahead.
// The body of a chunk is straight-line code (static taps, static register
// rings), so the loads of the next steps and of the next chunk stay in flight
// behind the matrix instructions; two tiles per compute unit cover each
// other's barriers.  The K-split partial sums are added in a fixed order
// through LDS, so the result does not depend on timing; P is then updated with
// 16-byte accesses.
// ---------------------------------------------------------------------------
template <int NSUB, int WMV, int WK, int TM, int TN, int KC, int NLD_, int KS, int RING_ = 3, int MINB_ = (NSUB >= 2 ? 2 : 1)>
struct HaloCfg {
    static constexpr int SUB = kSegPixels / NSUB;    // indices (and at most entries) per tile
    static_assert(WMV * WK == 4 && WMV * TM * 32 == SUB && SUB % 64 == 0, "4 waves cover one tile");
    static constexpr int BN = 32 * TN;
    static constexpr int KB = KC / 16;               // 16-channel blocks per chunk
    static_assert(KB % WK == 0, "every K wave takes the same number of blocks per tap");
    static constexpr int MB = KB / WK;               // blocks per tap and wave
    static constexpr int NS = KS * KS * MB;          // steps per chunk and wave
    static constexpr int RING = RING_;               // weight-fragment sets in flight; divides NS, so the
                                                     // ring carries over from chunk to chunk.  Above 3 the
                                                     // registers go to the ring and the next chunk of the
                                                     // rectangle is fetched at the chunk boundary instead of
                                                     // being prefetched into registers during the chunk
    static_assert(NS % RING == 0, "static ring slots");
    static constexpr int CPR = KC / 8;               // 16-byte pieces per staged pixel
    static constexpr int NLD = NLD_;                 // pieces per thread and chunk
    static constexpr int CAP = NLD * 256 / CPR;      // staged pixels
    static constexpr int LDK = KC + 8;               // staged row, halves (16 bytes of padding)
    static constexpr int LDC = BN + 4;               // accumulator row, floats
    static constexpr int HALO_BYTES = CAP * LDK * 2;
    static constexpr int C_BYTES = SUB * LDC * 4;
    // K-split partial sums: a buffer per K wave where that leaves room for two tiles per compute unit (one barrier, the
    // thread that updates P adds them up), else the waves take turns adding to one (a barrier per wave)
    static constexpr bool PARTS = WK > 1 && WK * C_BYTES <= 72 * 1024;
    static constexpr int SUM_BYTES = PARTS ? WK * C_BYTES : C_BYTES;
    static constexpr int MAIN_BYTES = HALO_BYTES > SUM_BYTES ? HALO_BYTES : SUM_BYTES;
    static constexpr int SMEM = MAIN_BYTES + (CAP + 2 * SUB + 8) * 4;   // + source pixel of every staged position, entries, counts
    static constexpr int LPS = (NLD + NS / 2 - 1) / (NS / 2);   // staging loads per step (first steps of a chunk)
    static constexpr int NLS = (NLD + LPS - 1) / LPS;
    static_assert(NLS <= NS, "staging loads fit the steps of a chunk");
    static constexpr int MINB = MINB_;               // tiles per compute unit the registers are budgeted for
};

// T2D: the tiles are th x tw rectangles of the padded window (th * tw <= SUB) instead of index ranges: the staged rectangle
// is the tile plus its KS - 1 halo whatever the width of the window, so wide rows fit and narrow ones stage less.
template <int NSUB, int WMV, int WK, int TM, int TN, int KC, int NLD_, int KS, int RING_ = 3, int MINB_ = (NSUB >= 2 ? 2 : 1), bool T2D = false>
__device__ __forceinline__ void halo_body(const EdgeDev& e, unsigned blk, unsigned nblk, int NT, int work_items, int th, int tw) {
    using Cfg = HaloCfg<NSUB, WMV, WK, TM, TN, KC, NLD_, KS, RING_, MINB_>;
    constexpr int SUB = Cfg::SUB, BN = Cfg::BN, KB = Cfg::KB, MB = Cfg::MB, NS = Cfg::NS, CPR = Cfg::CPR, NLD = Cfg::NLD,
                  LDK = Cfg::LDK, LDC = Cfg::LDC;
    constexpr bool PARTS = Cfg::PARTS;
    // Quarter-segment rectangles, which a launch has few of: what a tile can ask for before it knows what it needs goes out
    // at once - the first weight fragments, the rows of the rectangle whether updated or not, then the pending rows - so
    // that its round trips to memory overlap.  (Larger tiles fill the chip: there the same only adds traffic and registers.)
    constexpr bool EARLY = T2D && NSUB == 4;
    extern __shared__ __align__(16) unsigned char smem[];
    f16* halo = reinterpret_cast<f16*>(smem);            // [CAP][LDK] during the K loop
    float* sC = reinterpret_cast<float*>(smem);          // [SUB][LDC] after it
    int* s_pix = reinterpret_cast<int*>(smem + Cfg::MAIN_BYTES);
    int *const s_wy = s_pix + Cfg::CAP, *const s_wx = s_wy + SUB, *const sh = s_wx + SUB;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // wave-uniform: scalar branches below
    const int wm = wave % WMV, wk = wave / WMV;
    const int r32 = lane & 31, kh = lane >> 5;
    const int tiles_x = T2D ? (e.Wp + tw - 1) / tw : 1;
    const int ntiles = T2D ? tiles_x * ((e.Hp + th - 1) / th) : edge_segments(e) * NSUB;
    const int nchunks = e.Cin / KC;
    const int nwin = e.Hp * e.Wp;
    // (the host checks that both tensors are smaller than 2 GiB)
    const rsrc_t drs = make_rsrc(e.delta, (unsigned)e.sH * (unsigned)e.sW * (unsigned)e.Cin * 2u);
    const rsrc_t wrs = make_rsrc(e.wp, (unsigned)(KS * KS) * (unsigned)e.Cin * (unsigned)e.Cout * 2u);
    const unsigned tap_stride = (unsigned)(e.Cin / 16) * (unsigned)e.Cout * 32u;   // packed weights: bytes per tap
    const unsigned blk_stride = (unsigned)e.Cout * 32u;                            //                 per 16-channel block

    unsigned warm = 0;
    if constexpr (T2D) {
        static_assert(KS == 3, "what publish_edge takes: 3 x 3 and 1 x 1 edges");
        // the blocks of a cout tile touch that tile's weights, a line each, before anything else: the fragments of the
        // K loop then come from the L2 of their XCD instead of following each other to memory
        if constexpr (!EARLY) {
        const unsigned nt0 = blk % NT, sharers = nblk / NT > 0 ? nblk / NT : 1, rank = blk / NT;
        const unsigned kb = e.Cin / 16, lpf = BN * 32 / 128, nlines = KS * KS * kb * lpf;
        for (unsigned l = rank * 256 + tid; l < nlines; l += sharers * 256) {
            const unsigned f = l / lpf, ln = l - f * lpf, t = (unsigned)fast_div((int)f, (int)kb, rcp_of((int)kb));
            const unsigned off = t * tap_stride + (f - t * kb) * blk_stride + nt0 * BN * 32 + ln * 128;
            warm ^= (unsigned)__builtin_amdgcn_raw_buffer_load_b32(wrs, (int)off, 0, 0);
        }
        }
    } else {
        carry_source_compaction(e, sh, blk, nblk);
    }

    for (int u = (int)blk; u < work_items; u += (int)nblk) {
        const int nt = u % NT, mt = u / NT;              // u % 8 picks the XCD: few cout tiles per XCD
        if (mt >= ntiles) continue;
        const int n0 = nt * BN;
        const unsigned wlane = (unsigned)(r32 * 16 + kh * 8) * 2u;                      // this lane's bytes within a fragment
        const unsigned wwave = ((unsigned)wk * (unsigned)e.Cout + (unsigned)n0) * 32u;   // this wave's K block and cout tile
        f16x8 fa[Cfg::RING][TN];                          // weight fragments in flight
        auto load_a = [&](int slot, int c, int i) {       // step i of chunk c; i may run into the next chunk
            const int cc = i < NS ? c : (c + 1 < nchunks ? c + 1 : c), ii = i < NS ? i : i - NS;
            const unsigned src = wwave + (unsigned)(ii / MB) * tap_stride + (unsigned)(cc * KB + WK * (ii % MB)) * blk_stride;
#pragma unroll
            for (int j = 0; j < TN; ++j) fa[slot][j] = buf_load16(wrs, wlane, src + (unsigned)j * 32u * 32u);
        };
        if constexpr (EARLY) {
#pragma unroll
            for (int i = 0; i < Cfg::RING - 1; ++i) load_a(i, 0, i);
        }
        __syncthreads();                                  // previous tile is done with LDS
        int tot, wyA, wyB, cxA, cxB;                      // entries; window rows and source columns the tile spans
        f16x8 hreg[NLD];                                  // rows of the rectangle on their way to LDS
        constexpr int NRF = (Cfg::CAP + 255) / 256;       // rectangle positions per thread
        if constexpr (T2D) {
            const int ty = mt / tiles_x, tx = mt - ty * tiles_x;
            wyA = ty * th;
            wyB = (wyA + th < e.Hp ? wyA + th : e.Hp) - 1;
            cxA = tx * tw - e.bx0;
            cxB = (tx * tw + tw < e.Wp ? tx * tw + tw : e.Wp) - 1 - e.bx0;
            const int ry0 = wyA - e.by0 - e.pad, rx0 = cxA - e.pad, rw = cxB - cxA + KS, rn = (wyB - wyA + KS) * rw;
            const float rrw = rcp_of(rw);
            // the rectangle: source pixel of every position, -1 where it is out of view or not updated
            int rpix[NRF];
            unsigned rflag[NRF];
#pragma unroll
            for (int j = 0; j < NRF; ++j) {
                const int pos = tid + 256 * j;
                const int ry = fast_div(pos, rw, rrw), iy = ry0 + ry, ix = rx0 + pos - ry * rw;
                const bool ok = pos < rn && iy >= 0 && iy < e.sH && ix >= 0 && ix < e.sW;
                rpix[j] = ok ? iy * e.sW + ix : -1;
                rflag[j] = e.sflags[ok ? rpix[j] : 0];
            }
            if constexpr (EARLY) {
#pragma unroll
                for (int j = 0; j < NLD; ++j) {
                    const int q = tid + 256 * j, pos = q / CPR;
                    const int ry = fast_div(pos, rw, rrw), iy = ry0 + ry, ix = rx0 + pos - ry * rw;
                    const bool ok = pos < rn && iy >= 0 && iy < e.sH && ix >= 0 && ix < e.sW;
                    hreg[j] = buf_load16(drs, ok ? ((unsigned)(iy * e.sW + ix) * (unsigned)e.Cin + (q % CPR) * 8) * 2u : 0x80000000u, 0u);
                }
            }
#pragma unroll
            for (int j = 0; j < NRF; ++j) {
                const int pos = tid + 256 * j;
                if (pos < rn) s_pix[pos] = rpix[j] >= 0 && (rflag[j] & kFlagM) ? rpix[j] : -1;
            }
            __syncthreads();
            tot = tile_prologue_2d(e, ty * th, tx * tw, th, tw, s_pix, rw, s_wy, s_wx, sh);
        } else {
            const int seg = mt / NSUB, sub_lo = (mt % NSUB) * SUB;
            tot = tile_prologue_sub(e, seg, sub_lo, SUB, nt == 0 && sub_lo == 0, nt == 0, s_wy, s_wx, sh);
            // the source rectangle this index range reads (block-uniform)
            const int a = seg * kSegPixels + sub_lo;
            const int last = (a + SUB < nwin ? a + SUB : nwin) - 1;
            wyA = a / e.Wp; wyB = last / e.Wp;
            cxA = wyA == wyB ? a - wyA * e.Wp - e.bx0 : -e.bx0;
            cxB = wyA == wyB ? last - wyA * e.Wp - e.bx0 : e.Wp - 1 - e.bx0;
        }
        if (tot <= 0) continue;
        if (!T2D && tid == 0 && nt == 0) add_macs(e, sh[4], 0);
        const int iy0 = wyA - e.by0 - e.pad, ix0 = cxA - e.pad;
        const int RW = cxB - cxA + KS, npos = (wyB - wyA + KS) * RW;       // npos <= CAP: checked by the host
        if constexpr (!T2D) {                             // (rectangular tiles: s_pix was filled ahead of the prologue)
            for (int pos = tid; pos < npos; pos += 256) {
                const int ry = pos / RW, rx = pos - ry * RW;
                const int iy = iy0 + ry, ix = ix0 + rx;
                const bool ok = iy >= 0 && iy < e.sH && ix >= 0 && ix < e.sW && (e.sflags[iy * e.sW + ix] & kFlagM);
                s_pix[pos] = ok ? iy * e.sW + ix : -1;
            }
            __syncthreads();
        }
        const int nrt = (tot + 31) >> 5;                  // live 32-entry row tiles of the tile
        const int mylive = nrt > wm ? (nrt - wm + WMV - 1) / WMV : 0;      // of this wave: row tiles wm, wm + WMV, ...

        // staging: piece q = tid + 256 j is 16 bytes of staged pixel q / CPR (q / CPR < CAP: inside the buffer).
        // Dead pieces (outside the rectangle, out of view, not updated) are loaded from beyond the end of the
        // delta map, which a buffer load answers with zeros, and stored like the others: no predicates.
        unsigned hsrc[NLD];                               // byte offsets into the delta map
#pragma unroll
        for (int j = 0; j < NLD; ++j) {
            const int q = tid + 256 * j, pos = q / CPR;
            const int pix = pos < npos ? s_pix[pos] : -1;
            hsrc[j] = pix >= 0 ? ((unsigned)pix * (unsigned)e.Cin + (q % CPR) * 8) * 2u : 0x80000000u;
        }
        auto halo_store = [&]() {
#pragma unroll
            for (int j = 0; j < NLD; ++j) {
                const int q = tid + 256 * j;
                *reinterpret_cast<f16x8*>(halo + (q / CPR) * LDK + (q % CPR) * 8) = hreg[j];
            }
        };
#pragma unroll
        for (int j = 0; j < NLD; ++j) {
            if constexpr (EARLY) {
                if (hsrc[j] == 0x80000000u) hreg[j] = f16x8{};      // requested above, but not updated
            } else {
                hreg[j] = buf_load16(drs, hsrc[j], 0u);
            }
        }
        halo_store();

        f32x16 acc[TM][TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
        int rowoff[TM];                                   // this lane's staged row per row tile (halves)
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int r = (i * WMV + wm) * 32 + r32;
            rowoff[i] = kh * 8 + wk * 16 + (r < tot ? ((s_wy[r] - e.by0 - e.pad - iy0) * RW + (s_wx[r] - e.bx0 - e.pad - ix0)) * LDK : 0);
        }
        __syncthreads();

        // the pending rows this thread updates: all reads go out together (before the K loop where registers allow)
        constexpr int TPR = BN / 8;                        // threads per entry, 8 couts each
        constexpr int RPP = 256 / TPR, NPASS = (SUB + RPP - 1) / RPP;
        const int c8 = (tid % TPR) * 8;
        f16x8 pold[NPASS];
        f16* pp[NPASS];
        auto load_p = [&] {
#pragma unroll
            for (int t = 0; t < NPASS; ++t) {
                const int row = tid / TPR + t * RPP;
                const int rr = row < tot ? row : 0;         // dead rows read entry 0 and store nothing
                pp[t] = (f16*)e.P + pdst_offset(e, s_wy[rr], s_wx[rr]) + n0 + c8;
                pold[t] = *reinterpret_cast<const f16x8*>(pp[t]);
            }
        };
        if constexpr (EARLY) load_p();

        // The K loop for L live row tiles of this wave.  Step i of a chunk: tap i / MB,
        // 16-channel block wk + WK * (i % MB) of the chunk.
        auto kloop = [&](auto lc) {
            constexpr int L = decltype(lc)::value;
            constexpr int D = Cfg::RING;
            constexpr int FBR = TM > 4 ? 2 : 3;                      // sets of staged-row fragments in flight
            f16x8 fb[FBR][L > 0 ? L : 1];
            auto load_b = [&](int slot, int i) {
                const int tap = i / MB;
                const f16* hb = halo + ((tap / KS) * RW + tap % KS) * LDK + WK * (i % MB) * 16;
#pragma unroll
                for (int t = 0; t < L; ++t) fb[slot][t] = *reinterpret_cast<const f16x8*>(hb + rowoff[t]);
            };
            if constexpr (!EARLY) {
#pragma unroll
                for (int i = 0; i < D - 1; ++i) load_a(i, 0, i);
            }
            for (int c = 0; c < nchunks; ++c) {
                const int cn = c + 1 < nchunks ? c + 1 : c;          // the last chunk re-reads itself: no branch
                const unsigned hc = (unsigned)cn * KC * 2u;
#pragma unroll
                for (int i = 0; i < FBR - 1; ++i) load_b(i, i);
#pragma unroll
                for (int i = 0; i < NS; ++i) {
                    if (Cfg::RING <= 3 && i < Cfg::NLS) { // staging loads of the next chunk, a few per step
#pragma unroll
                        for (int j = i * Cfg::LPS; j < (i + 1) * Cfg::LPS && j < NLD; ++j)
                            hreg[j] = buf_load16(drs, hsrc[j], hc);
                    }
                    load_a((i + D - 1) % D, c, i + D - 1);
                    if (i + FBR - 1 < NS) load_b((i + FBR - 1) % FBR, i + FBR - 1);
#pragma unroll
                    for (int t = 0; t < L; ++t)
#pragma unroll
                        for (int j = 0; j < TN; ++j)
                            acc[t][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[i % D][j], fb[i % FBR][t], acc[t][j], 0, 0, 0);
                    // the loads just issued (for later steps) stay ahead of these MFMAs and are
                    // spread between them: one LDS read, one global load, a quarter of the MFMAs
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                       // one LDS read
                        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);                       // one global load
                        __builtin_amdgcn_sched_group_barrier(0x008, (L * TN + 3) / 4, 0);        // a quarter of the MFMAs
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                __syncthreads();                          // everyone is done reading the staged chunk
                if (c + 1 < nchunks) {
                    if constexpr (Cfg::RING > 3) {        // deep weight ring: the registers go to it, the next chunk is
                                                          // fetched here (the weight loads of its first steps are in flight)
#pragma unroll
                        for (int j = 0; j < NLD; ++j) hreg[j] = buf_load16(drs, hsrc[j], hc);
                    }
                    halo_store();
                    __syncthreads();
                }
            }
        };
        if constexpr (EARLY) kloop(std::integral_constant<int, TM>{});     // (a second loop body would not share the ring's registers)
        else switch (mylive) {
            case 0: kloop(std::integral_constant<int, 0>{}); break;
            case 1: kloop(std::integral_constant<int, 1>{}); break;
            case 2: kloop(std::integral_constant<int, TM >= 2 ? 2 : TM>{}); break;
            case 3: kloop(std::integral_constant<int, (TM > 4 ? 4 : TM >= 3 ? 3 : TM)>{}); break;    // rounded up: dead tiles are not stored
            case 4: kloop(std::integral_constant<int, (TM >= 4 ? 4 : TM)>{}); break;
            default: kloop(std::integral_constant<int, TM>{}); break;
        }

        if constexpr (!EARLY) load_p();
        // K-split partial sums -> LDS [entry][cout], a buffer per K wave or added up in turns; either way every element
        // is added up in the order of the K waves.
        auto put = [&](int i, bool add) {
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                float* dst = sC + (PARTS ? wk * SUB * LDC : 0) + ((i * WMV + wm) * 32 + r32) * LDC + j * 32 + 4 * kh;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    float4 v = make_float4(acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
                    if (add) {
                        const float4 o = *reinterpret_cast<const float4*>(dst + 8 * g);
                        v.x += o.x; v.y += o.y; v.z += o.z; v.w += o.w;
                    }
                    *reinterpret_cast<float4*>(dst + 8 * g) = v;
                }
            }
        };
        if constexpr (PARTS) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
                if (i < mylive) put(i, false);
            __syncthreads();
        } else {
#pragma unroll
            for (int kq = 0; kq < WK; ++kq) {
                if (wk == kq) {
#pragma unroll
                    for (int i = 0; i < TM; ++i)
                        if (i < mylive) put(i, kq > 0);
                }
                __syncthreads();
            }
        }
        // P <- P + sum
#pragma unroll
        for (int t = 0; t < NPASS; ++t) {
            const int row = tid / TPR + t * RPP;
            if (row < tot) {
                float v[8];
#pragma unroll
                for (int kq = 0; kq < (PARTS ? WK : 1); ++kq) {
                    const float* src = sC + kq * SUB * LDC + row * LDC + c8;
                    const float4 v0 = *reinterpret_cast<const float4*>(src), v1 = *reinterpret_cast<const float4*>(src + 4);
                    const float part[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
#pragma unroll
                    for (int q = 0; q < 8; ++q) v[q] = kq ? v[q] + part[q] : part[q];
                }
                f16x8 o = pold[t];
#pragma unroll
                for (int q = 0; q < 8; ++q) o[q] = (f16)((float)o[q] + v[q]);
                *reinterpret_cast<f16x8*>(pp[t]) = o;
            }
        }
    }
    if (warm == 0x9e3779b9u && work_items < 0) e.ccnt[0] = 0;     // (keeps the loads above)
}

}  // namespace mdcnn
