// Padded sparse convolution: for every entry of the compute list (a pixel of
// the destination's padded window whose footprint holds an updated input pixel)
//   y[q, :] = sum over taps with an updated in-view input  W[tap] . delta[p(q, tap), :]
//   P_dst[q] <- P_dst[q] + y[q]        (border pixels included: they are stashed)
// Output-stationary: one owner per output pixel, fixed summation order, so the
// result does not depend on scheduling.  Weights are w[tap][cout][cin].
// There is no separate list kernel: every block finds the entries of its own tile from the source's update mask.  The lists
// the ABI exposes, the touched marks and the counts of a 3x3 or 1x1 edge on the matrix cores, of a 3-channel stem and of a
// residual skip are left to a few blocks at the end of the launch (publish_edge), and where the destination is an OUTPUT site
// that a frame call reads out, blocks behind those copy what the tiles leave alone (read_rest).  The other kernels, and edges
// of other sizes, do it themselves: the block of a segment's first piece writes the segment (kSegPixels indices, one per
// thread, ballot + popcount ranks) to the compute list, and every block compacts its share of the source's mask into L.
//
//   k_conv_rect       : 3x3 fp16 layers with packed weights, stride 1 and 64 n input channels or stride 2 and
//                       32 n: rectangles, staged by loads that write LDS themselves, packed weights straight into
//                       MFMA fragments (conv_rect.h)
//   k_conv_halo       : the other 3x3 stride-1 fp16 layers of 32 n input channels: rectangles, staged
//                       through registers once per 32 channels
//   k_conv_mfma_tiled : LDS-tiled gather-GEMM on the CDNA4 matrix cores (fp16 in, fp32 acc): 1x1 and upsampling
//                       edges, strides above 2, layers without packed weights
//   k_conv_mfma_f16   : MFMA without LDS staging (fallback for Cin % 32 != 0)
//   k_conv_mfma_f32   : small fp32 layers, weights in LDS (fp32 matrix instruction)
//   k_conv_f32        : weights and delta rows staged in LDS (conv_f32.h): all other fp32 layers with
//                       Cin % 8 == 0 and Cout 16 or a multiple of 32, but for the smallest (f32_applies)
//   k_conv_stem_mfma  : 3-channel 3x3 stems on the fp32 matrix instruction
//   k_conv_small      : 3-channel 3x3 stems, plain FMA (upsampling edges and where the matrix cores are switched off)
//   k_conv_ldsw       : plain FMA with the weights resident in LDS (fp32 layers of few products, other shapes)
//   k_conv_plain      : plain FMA, any dtype / channel count
//   k_identity        : residual skip, P_dst[q] += delta[q] (when it is not fused into step 1)
//   k_pool            : max pooling in delta form against a previous-output ring
//   k_pack_weights    : [tap][cout][cin] -> [tap][cin/16][cout][16]
#include <atomic>
#include <mutex>
#include <type_traits>

#include "conv_rect.h"
#include "conv_tiles.h"
#include "conv_up.h"

namespace mdcnn {

static unsigned cap_blocks(long long b, long long cap) {
    if (b < 1) b = 1;
    if (b > cap) b = cap;
    return (unsigned)b;
}

// One edge per launch (blockIdx.z: stream of the batch); the tiles are those of conv_tiles.h.
template <int WM, int WN, int TM, int TN, int KC, int PIPE>
__global__ __launch_bounds__(256, (TiledCfg<WM, WN, TM, TN, KC, PIPE>::WAVES)) void k_conv_mfma_tiled(TileGrid g, unsigned blocks, int work_items, EdgeBatch eb) {
    extern __shared__ __align__(16) unsigned char smem[];
    const unsigned nblk = blocks - g.npub - g.ncopy;
    if (blockIdx.x >= nblk) side_block<f16>(eb.d[blockIdx.z], g, blockIdx.x - nblk, smem);
    else tiled_body<WM, WN, TM, TN, KC, PIPE, true>(eb.d[blockIdx.z], blockIdx.x, nblk, g, work_items);
}
template <int NSUB, int WMV, int WK, int TM, int TN, int KC, int NLD_, int KS, int RING_ = 3, int MINB_ = (NSUB >= 2 ? 2 : 1), bool T2D = false>
__global__ __launch_bounds__(256, MINB_) void k_conv_halo(EdgeBatch eb, unsigned npub, int NT, int work_items, int th, int tw) {
    const unsigned nblk = gridDim.x - npub;
    if (blockIdx.x >= nblk) publish_edge(eb.d[blockIdx.z], blockIdx.x - nblk, npub);
    else halo_body<NSUB, WMV, WK, TM, TN, KC, NLD_, KS, RING_, MINB_, T2D>(eb.d[blockIdx.z], blockIdx.x, nblk, NT, work_items, th, tw);
}

template <typename Cfg>
__global__ __launch_bounds__(256, Cfg::MINB) void k_conv_rect(TileGrid g, unsigned blocks, EdgeBatch eb) {
    extern __shared__ __align__(16) unsigned char smem[];
    const unsigned nblk = blocks - g.npub - g.ncopy;
    if (blockIdx.x >= nblk) side_block<f16>(eb.d[blockIdx.z], g, blockIdx.x - nblk, smem);
    else rect_body<Cfg, true>(eb.d[blockIdx.z], blockIdx.x, g);
}

__global__ __launch_bounds__(256) void k_conv_up(TileGrid g, unsigned blocks, EdgeBatch eb) {
    extern __shared__ __align__(16) unsigned char smem[];
    const unsigned nblk = blocks - g.npub - g.ncopy;
    if (blockIdx.x >= nblk) side_block<f16>(eb.d[blockIdx.z], g, blockIdx.x - nblk, smem);
    else up_body<true>(eb.d[blockIdx.z], blockIdx.x, g);
}

// Weights [tap][cout][cin] -> [tap][cin/16][cout][16]: the 32 couts x 16 cin
// operand of one MFMA becomes 1 KiB of consecutive memory.  One thread per 8 halves.
__global__ __launch_bounds__(256) void k_pack_weights(const f16* __restrict__ src, f16* __restrict__ dst, int taps, int Cout, int Cin) {
    const long long n8 = (long long)taps * Cout * Cin / 8;
    const int KBT = Cin / 16;
    for (long long i = blockIdx.x * 256ll + threadIdx.x; i < n8; i += gridDim.x * 256ll) {
        const int h = (int)(i & 1);
        long long r = i >> 1;
        const int co = (int)(r % Cout); r /= Cout;
        const int kb = (int)(r % KBT);
        const int tap = (int)(r / KBT);
        *reinterpret_cast<f16x8*>(dst + i * 8) =
            *reinterpret_cast<const f16x8*>(src + ((long long)tap * Cout + co) * Cin + kb * 16 + h * 8);
    }
}

// ---------------------------------------------------------------------------
// MFMA without LDS staging: every wave loads its own fragments from global
// memory.  Block = 4 waves arranged (4/WN) x WN over (pixels x couts); every
// lane updates its own pixel of P.  Fallback for Cin % 32 != 0.
// ---------------------------------------------------------------------------
template <int WN>
__global__ __launch_bounds__(256) void k_conv_mfma_f16(EdgeBatch eb) {
    const EdgeDev& e = eb.d[blockIdx.z];                  // blockIdx.z: stream of the batch
    constexpr int WM = 4 / WN;
    constexpr int TILE_M = 32 * WM;
    constexpr int TPS = kSegPixels / TILE_M;
    __shared__ int s_base[TILE_M], s_wy[TILE_M], s_wx[TILE_M];
    __shared__ unsigned s_vm[TILE_M];
    __shared__ int sh[8];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave % WM, wn = wave / WM;
    const int col = lane & 31, kh = lane >> 5;
    const int MT = edge_segments(e) * TPS;
    const int n0 = (blockIdx.y * WN + wn) * 32;
    const f16* __restrict__ delta = (const f16*)e.delta;
    const f16* __restrict__ w = (const f16*)e.w;
    const int taps = e.k * e.k;
    carry_source_compaction(e, sh);
    for (int tile = blockIdx.x; tile < MT; tile += gridDim.x) {
        const int seg = tile / TPS, first = (tile - seg * TPS) * TILE_M;
        __syncthreads();
        const int tot = tile_prologue(e, seg, first, TILE_M, blockIdx.y == 0 && first == 0 && !e.up, blockIdx.y == 0,
                                      s_base, s_wy, s_wx, s_vm, sh);
        if (first >= tot) continue;
        if (threadIdx.x == 0 && blockIdx.y == 0) add_macs(e, sh[4], 0);
        const int row = wm * 32 + col;
        const bool live = first + row < tot;
        const unsigned vmask = s_vm[row];
        const int base = s_base[row], wy = s_wy[row], wx = s_wx[row];
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
        for (int tap = 0; tap < taps; ++tap) {
            const bool v = (vmask >> tap) & 1u;
            if (__ballot(v) == 0ull) continue;                 // no pixel of this wave uses the tap
            const int jy = tap / e.k, jx = tap - jy * e.k;
            const f16* arow = w + ((size_t)(tap * e.Cout + n0 + col)) * e.Cin + kh * 8;
            const f16* brow = delta + (v ? ((size_t)(base + jy * e.sW + jx)) * e.Cin + kh * 8 : 0);
            for (int c0 = 0; c0 < e.Cin; c0 += 16) {
                f16x8 a = *reinterpret_cast<const f16x8*>(arow + c0);
                f16x8 b;
                if (v) b = *reinterpret_cast<const f16x8*>(brow + c0);
                else {
#pragma unroll
                    for (int i = 0; i < 8; ++i) b[i] = (f16)0.f;
                }
                acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, acc, 0, 0, 0);
            }
        }
        if (live) {
            const int f = 1 << e.up;
            for (int ua = 0; ua < f; ++ua)
                for (int ub = 0; ub < f; ++ub) {
                    f16* p = (f16*)e.P + pdst_offset(e, wy + ua, wx + ub) + n0 + 4 * kh;
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        f16x4 o = *reinterpret_cast<f16x4*>(p + 8 * g);
#pragma unroll
                        for (int i = 0; i < 4; ++i) o[i] = (f16)((float)o[i] + acc[4 * g + i]);
                        *reinterpret_cast<f16x4*>(p + 8 * g) = o;
                    }
                }
        }
    }
}

template <typename T> struct Row8;
template <> struct Row8<f16> {
    typedef f16x8 reg;                                      // eight stored values, fetched ahead of their use
    __device__ static reg load(const f16* p) { return *reinterpret_cast<const f16x8*>(p); }
    __device__ static void add_store(f16* p, reg o, const float* v) {
#pragma unroll
        for (int q = 0; q < 8; ++q) o[q] = (f16)((float)o[q] + v[q]);
        *reinterpret_cast<f16x8*>(p) = o;
    }
    __device__ static void add(f16* p, const float* v) { add_store(p, load(p), v); }
};
template <> struct Row8<float> {
    struct reg { float4 a, b; };
    __device__ static reg load(const float* p) { return reg{*reinterpret_cast<const float4*>(p), *reinterpret_cast<const float4*>(p + 4)}; }
    __device__ static void add_store(float* p, reg o, const float* v) {
        o.a.x += v[0]; o.a.y += v[1]; o.a.z += v[2]; o.a.w += v[3];
        o.b.x += v[4]; o.b.y += v[5]; o.b.z += v[6]; o.b.w += v[7];
        *reinterpret_cast<float4*>(p) = o.a;
        *reinterpret_cast<float4*>(p + 4) = o.b;
    }
    __device__ static void add(float* p, const float* v) { add_store(p, load(p), v); }
};

// ---------------------------------------------------------------------------
// Plain FMA convolution with ALL weights resident in LDS as fp32
// [tap][cin][cout]; a thread owns one list entry and 8 consecutive couts.
// Used for fp32 networks and for layers the MFMA path does not take (e.g. a
// 3-channel stem).  Needs Cout % 8 == 0, Cout <= 512 and k*k*Cin*Cout*4 bytes
// of LDS.  Tiles of ppb entries never straddle a list segment.
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void k_conv_ldsw(EdgeBatch eb, int groups, int ppb) {
    const EdgeDev& e = eb.d[blockIdx.z];                  // blockIdx.z: stream of the batch
    extern __shared__ __align__(16) unsigned char smem[];
    float* sW = reinterpret_cast<float*>(smem);             // [tap][Cin][Cout]
    __shared__ int s_base[256], s_wy[256], s_wx[256];
    __shared__ unsigned s_vm[256];
    __shared__ int sh[8];
    const int tid = threadIdx.x;
    const int cg = tid % groups, pl = tid / groups;         // cout group, local pixel
    const T* __restrict__ delta = (const T*)e.delta;
    const T* __restrict__ w = (const T*)e.w;
    const int taps = e.k * e.k;
    const int cc = e.Cin * e.Cout;
    carry_source_compaction(e, sh);
    // weights [tap][cout][cin] -> LDS [tap][cin][cout] as fp32.  Neighbouring threads take neighbouring couts, so
    // their LDS stores fall into different banks; a thread reads 16 bytes of its weight row at a time.
    constexpr int WV = 16 / (int)sizeof(T);
    if (e.Cin % WV == 0) {
        // Eight reads of a thread are in flight at a time (the copy is a chain of round trips otherwise, and it is
        // the larger part of a launch on sparse frames); a read past the end of the tensor returns zeros and is dropped.
        const int pieces = e.Cin / WV, total = taps * pieces * e.Cout;
        const rsrc_t wrs = make_rsrc(w, (unsigned)(taps * cc) * (unsigned)sizeof(T));
        constexpr int WU = 8;
        for (int i0 = tid; i0 < total; i0 += 256 * WU) {
            u32x4_t raw[WU];
            int dst[WU];
#pragma unroll
            for (int u = 0; u < WU; ++u) {
                const int i = i0 + u * 256;
                const int co = i % e.Cout, q = i / e.Cout;
                const int piece = q % pieces, tap = q / pieces;
                const bool in = i < total;
                dst[u] = in ? tap * cc + piece * WV * e.Cout + co : -1;
                raw[u] = __builtin_amdgcn_raw_buffer_load_b128(
                    wrs, in ? (int)(((unsigned)(tap * e.Cout + co) * (unsigned)e.Cin + (unsigned)(piece * WV)) * (unsigned)sizeof(T)) : (int)0x80000000u, 0, 0);
            }
#pragma unroll
            for (int u = 0; u < WU; ++u) {
                if (dst[u] < 0) continue;
                T a[WV];
                __builtin_memcpy(a, &raw[u], 16);
#pragma unroll
                for (int v = 0; v < WV; ++v) sW[dst[u] + v * e.Cout] = (float)a[v];
            }
        }
    } else {
        for (int i = tid; i < taps * cc; i += 256) {
            const int tap = i / cc, r = i - tap * cc;
            const int co = r / e.Cin, ci = r - co * e.Cin;
            sW[tap * cc + ci * e.Cout + co] = (float)w[i];
        }
    }
    long long block_taps = 0;                               // statistics (thread 0 only)
    const int tps = (kSegPixels + ppb - 1) / ppb;           // tiles per segment
    const int MT = edge_segments(e) * tps;
    for (int tile = blockIdx.x; tile < MT; tile += gridDim.x) {
        const int seg = tile / tps, first = (tile - seg * tps) * ppb;
        __syncthreads();
        const int tot = tile_prologue(e, seg, first, ppb, first == 0 && !e.up, true, s_base, s_wy, s_wx, s_vm, sh);
        if (first >= tot) continue;
        if (tid == 0) block_taps += sh[4];
        if (pl >= ppb || first + pl >= tot) continue;
        const unsigned vmask = s_vm[pl];
        const int base = s_base[pl];
        float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (int tap = 0; tap < taps; ++tap) {
            if (!((vmask >> tap) & 1u)) continue;
            const int jy = tap / e.k, jx = tap - jy * e.k;
            const T* drow = delta + (size_t)(base + jy * e.sW + jx) * e.Cin;
            const float* wt = sW + tap * cc + cg * 8;
            auto mac = [&](float a, int ci) {               // channels in ascending order: the sum does not change
                const float4 w0 = *reinterpret_cast<const float4*>(wt + ci * e.Cout);
                const float4 w1 = *reinterpret_cast<const float4*>(wt + ci * e.Cout + 4);
                acc[0] = fmaf(a, w0.x, acc[0]); acc[1] = fmaf(a, w0.y, acc[1]);
                acc[2] = fmaf(a, w0.z, acc[2]); acc[3] = fmaf(a, w0.w, acc[3]);
                acc[4] = fmaf(a, w1.x, acc[4]); acc[5] = fmaf(a, w1.y, acc[5]);
                acc[6] = fmaf(a, w1.z, acc[6]); acc[7] = fmaf(a, w1.w, acc[7]);
            };
            constexpr int V = 16 / (int)sizeof(T);           // a row is read in 16-byte pieces, several of them in flight
            if (e.Cin % V == 0) {
#pragma unroll 8
                for (int ci = 0; ci < e.Cin; ci += V) {
                    const u32x4_t raw = *reinterpret_cast<const u32x4_t*>(drow + ci);
                    T a[V];
                    __builtin_memcpy(a, &raw, 16);
#pragma unroll
                    for (int v = 0; v < V; ++v) mac((float)a[v], ci + v);
                }
            } else {
                for (int ci = 0; ci < e.Cin; ++ci) mac((float)drow[ci], ci);
            }
        }
        const int f = 1 << e.up;
        for (int ua = 0; ua < f; ++ua)
            for (int ub = 0; ub < f; ++ub)
                Row8<T>::add((T*)e.P + pdst_offset(e, s_wy[pl] + ua, s_wx[pl] + ub) + cg * 8, acc);
    }
    if (tid == 0) add_macs(e, block_taps, 1);               // statistics: one atomic per block
}

// ---------------------------------------------------------------------------
// fp32 layers on the matrix cores (v_mfma_f32_32x32x2_f32), Cin and footprint at
// compile time, Cout 16 or a multiple of 32, no upsampling.  A block owns one tile of
// 32 couts (blockIdx.y) and keeps its weights in LDS as [tap][cin][32]; its four
// waves are 4 / KS groups of 32 list entries x KS shares of the taps (wave k
// of a group takes taps k, k + KS, ...), and the partial sums of a group are
// added through LDS in a fixed order.  The matrix instruction takes the couts
// as rows and the entries as columns: a lane holds entry lane % 32 and half
// lane / 32 of the K pair, which is channel (lane / 32) * CIN / 2 + step - so a
// lane reads CIN / 2 consecutive channels of its entry's source row per tap, in
// 16-byte pieces, one tap ahead of the multiplication, and one weight per
// instruction from LDS (32 consecutive floats per half wave).  Taps outside an
// entry's mask are read from beyond the end of the tensor (zeros); the tap loop
// has no branches.
// ---------------------------------------------------------------------------
template <int KK, int CIN, int KS>
__global__ __launch_bounds__(256) void k_conv_mfma_f32(unsigned npub, unsigned ncopy, unsigned blocks, EdgeBatch eb) {
    EdgeDev e = eb.d[blockIdx.z];                         // blockIdx.z: stream of the batch
    extern __shared__ __align__(16) unsigned char smem[];
    const unsigned nblk = blocks - npub - ncopy;
    if (blockIdx.x >= nblk) {
        if (blockIdx.y == 0) side_block<float>(e, TileGrid{npub, ncopy}, blockIdx.x - nblk, smem);
        return;
    }
    read_now(e.delta, e.sflags, e.sH, e.sW, e.P, e.Cout, e.Hp, e.Wp, e.by0, e.bx0, e.p_oy, e.p_ox, e.w, e.k, e.stride, e.pad, e.up, e.op);
    float* sW = reinterpret_cast<float*>(smem);             // [tap][CIN][32]
    constexpr int TAPS = KK * KK, HALF = CIN / 2, NP = HALF / 4, PGS = 4 / KS, BM = PGS * 32, NQ = (TAPS + KS - 1) / KS;
    constexpr int CC = CIN * 32;                            // floats per tap in LDS
    __shared__ int s_base[BM], s_wy[BM], s_wx[BM];
    __shared__ unsigned s_vm[BM];
    __shared__ int sh[8];
    __shared__ float s_red[KS > 1 ? PGS * (KS - 1) * 1024 : 1];    // partial sums of the waves that do not write P
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int p32 = lane & 31, h = lane >> 5;
    const int pg = wave % PGS, ks = wave / PGS;             // entry group, share of the taps
    const int nt = blockIdx.y;                              // cout tile
    const int ncout = e.Cout - nt * 32 < 32 ? e.Cout - nt * 32 : 32;      // 16 for a 16-cout layer: the other rows of the tile are not stored
    const float* __restrict__ w = (const float*)e.w;
    // weights [tap][cout][cin] -> LDS [tap][cin][32], eight 16-byte reads of a thread in flight.  The first eight are
    // requested here and stored after the prologue of the block's first tile, whose flag reads they travel with.
    constexpr int pieces = CIN / 4, WU = 8, wtotal = TAPS * pieces * 32;
    const rsrc_t wrs = make_rsrc(w, (unsigned)(TAPS * CIN) * (unsigned)e.Cout * 4u);
    auto request = [&](int i0, u32x4_t* raw, int* dst) {
#pragma unroll
        for (int u = 0; u < WU; ++u) {
            const int i = i0 + u * 256;
            const int co = i % 32, q = i / 32;
            const int piece = q % pieces, tap = q / pieces;
            const bool in = i < wtotal && co < ncout;
            dst[u] = in ? tap * CC + piece * 4 * 32 + co : -1;
            raw[u] = __builtin_amdgcn_raw_buffer_load_b128(
                wrs, in ? (int)(((unsigned)(tap * e.Cout + nt * 32 + co) * (unsigned)CIN + (unsigned)(piece * 4)) * 4u) : (int)0x80000000u, 0, 0);
        }
    };
    auto store = [&](const u32x4_t* raw, const int* dst) {
#pragma unroll
        for (int u = 0; u < WU; ++u) {
            if (dst[u] < 0) continue;
            float a[4];
            __builtin_memcpy(a, &raw[u], 16);
#pragma unroll
            for (int v = 0; v < 4; ++v) sW[dst[u] + v * 32] = a[v];
        }
    };
    u32x4_t raw0[WU];
    int dst0[WU];
    request(tid, raw0, dst0);
    bool weights_in = false;
    const rsrc_t drs = make_rsrc(e.delta, (unsigned)e.sH * (unsigned)e.sW * (unsigned)CIN * 4u);
    constexpr int TPS = kSegPixels / BM;                    // tiles per segment
    const int MT = edge_segments(e) * TPS;
    for (int tile = blockIdx.x; tile < MT; tile += (int)nblk) {
        const int seg = tile / TPS, first = (tile - seg * TPS) * BM;
        __syncthreads();
        const int tot = tile_prologue(e, seg, first, BM, false, false, s_base, s_wy, s_wx, s_vm, sh);
        if (!weights_in) {                                  // first tile of the block (block-uniform)
            store(raw0, dst0);
            for (int i0 = tid + 256 * WU; i0 < wtotal; i0 += 256 * WU) {
                u32x4_t raw[WU];
                int dst[WU];
                request(i0, raw, dst);
                store(raw, dst);
            }
            weights_in = true;
            __syncthreads();
        }
        if (first >= tot) continue;                         // block-uniform
        const bool wave_on = first + pg * 32 < tot;         // wave-uniform: the group has entries
        const int pl = pg * 32 + p32;
        const bool act = first + pl < tot;
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
        if (wave_on) {
            const unsigned vmask = act ? s_vm[pl] : 0u;
            const int rowb = act ? (s_base[pl] * CIN + h * HALF) * 4 : 0;  // bytes; negative for a border entry's first taps
            auto load_tap = [&](int tap, u32x4_t* r) {      // tap >= TAPS (the last round of some waves): zeros
                const bool v = tap < TAPS && ((vmask >> tap) & 1u);
                const int jy = tap / KK, jx = tap - jy * KK;
                const int tb = rowb + (jy * e.sW + jx) * CIN * 4;
#pragma unroll
                for (int i = 0; i < NP; ++i)
                    r[i] = __builtin_amdgcn_raw_buffer_load_b128(drs, v ? tb + i * 16 : (int)0x80000000u, 0, 0);
            };
            u32x4_t rows[2][NP];
            load_tap(ks, rows[0]);
            const float* wl = sW + h * HALF * 32 + p32;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int tap = ks + KS * q;
                if (q + 1 < NQ) load_tap(tap + KS, rows[(q + 1) & 1]);
                const float* wt = wl + (tap < TAPS ? tap : TAPS - 1) * CC;
#pragma unroll
                for (int i = 0; i < NP; ++i) {
                    float b[4];
                    __builtin_memcpy(b, &rows[q & 1][i], 16);
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wt[(i * 4 + j) * 32], b[j], acc, 0, 0, 0);
                }
            }
        }
        if constexpr (KS > 1) {
            if (wave_on && ks > 0) {
                float* red = s_red + (pg * (KS - 1) + ks - 1) * 1024 + lane;
#pragma unroll
                for (int r = 0; r < 16; ++r) red[r * 64] = acc[r];
            }
            __syncthreads();                                // all threads of the block, whatever their wave does
            if (wave_on && ks == 0) {
#pragma unroll
                for (int k = 1; k < KS; ++k) {
                    const float* red = s_red + (pg * (KS - 1) + k - 1) * 1024 + lane;
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[r] += red[r * 64];
                }
            }
        }
        // register r of a lane: cout 8 * (r / 4) + 4 * (lane / 32) + r % 4 of the tile, entry lane % 32
        if (act && ks == 0) {
            float* pp = (float*)e.P + pdst_offset(e, s_wy[pl], s_wx[pl]) + nt * 32 + 4 * h;
            float4 o[4];
#pragma unroll
            for (int g = 0; g < 4; ++g)
                if (8 * g < ncout) o[g] = *reinterpret_cast<const float4*>(pp + 8 * g);
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                if (8 * g >= ncout) continue;
                o[g].x += acc[4 * g]; o[g].y += acc[4 * g + 1]; o[g].z += acc[4 * g + 2]; o[g].w += acc[4 * g + 3];
                *reinterpret_cast<float4*>(pp + 8 * g) = o[g];
            }
            if (e.dY) {                                     // (the launch reads the site out)
                const int oy = s_wy[pl] - e.by0, ox = s_wx[pl] - e.bx0;
                if ((unsigned)oy < (unsigned)e.dH && (unsigned)ox < (unsigned)e.dW)
#pragma unroll
                    for (int g = 0; g < 4; ++g)
                        if (8 * g < ncout)
                            write_out<float, 4>((float*)e.dY, e.s_relu, ((size_t)oy * e.dW + ox) * e.Cout + nt * 32 + 4 * h + 8 * g, &o[g].x);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// 3x3 stems with 3 input channels on the matrix cores, fp32 or fp16 storage
// (fp16 values are exact in fp32, so both use v_mfma_f32_32x32x2_f32 with the
// weights as fp32 in LDS).  K = 27 products per output, padded to 28: lane half
// h of a wave holds k = 14 h + step, k = 9 jy + 3 jx + ci, which is element
// (k / 9) * 3 sW + k % 9 after the entry's first tap - the three pixels of a
// footprint row are nine consecutive values.  A block owns 128 list entries and
// one tile of 32 couts (blockIdx.y), a wave 32 entries; a lane fetches its 14
// values with single-element buffer loads that all go out together (a tap
// outside the entry's mask reads beyond the tensor: zero).  The lists, touched
// marks and counts are left to the last npub blocks (publish_edge): a stem's
// source has four times the pixels of its destination, and every tile used to
// compact its share of them, a round trip and two barriers per segment, before
// its own loads: 512 x 512 frames and 64 couts 15.4 -> 14.1 us, 384 x 288
// 12.4 -> 10.3, 256 x 256 fp32 and 32 couts 9.3 -> 7.6; boxes of 720 x 1280
// frames 29.5 either way.  What bounds it: the round trips of a tile, flags,
// deltas and pending rows.  (64 couts to a block with P updated through LDS in
// whole rows has half the blocks and is slower: 15.9 us, 33 on the boxes.)
// Five waves to a SIMD cover those round trips better than the four the
// compiler's own choice of registers (102) leaves: 512 x 512 frames of 16 videos
// 170 -> 161 us, of one 17.0 -> 16.6.
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256, 5) void k_conv_stem_mfma(unsigned npub, unsigned blocks, EdgeBatch eb) {
    EdgeDev e = eb.d[blockIdx.z];                         // blockIdx.z: stream of the batch
    const unsigned nblk = blocks - npub;
    if (blockIdx.x >= nblk) {
        if (blockIdx.y == 0) publish_edge(e, blockIdx.x - nblk, npub);
        return;
    }
    read_now(e.delta, e.sflags, e.sH, e.sW, e.P, e.Cout, e.Hp, e.Wp, e.by0, e.bx0, e.p_oy, e.p_ox, e.w, e.k, e.stride, e.pad, e.up, e.op);
    constexpr int BM = 128, KH = 14;
    __shared__ float sW[2 * KH * 32];                       // [k][32 couts], row 27 zero
    __shared__ int s_base[BM], s_wy[BM], s_wx[BM];
    __shared__ unsigned s_vm[BM];
    __shared__ int sh[8];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int p32 = lane & 31, h = lane >> 5;
    const int nt = blockIdx.y;
    const T* __restrict__ w = (const T*)e.w;
    for (int i = tid; i < 28 * 32; i += 256) {              // weights [tap][cout][3] -> LDS [k = 3 tap + ci][cout of the tile]
        const int k = i >> 5, co = i & 31;
        sW[i] = k < 27 ? (float)w[((k / 3) * e.Cout + nt * 32 + co) * 3 + k % 3] : 0.f;
    }
    const rsrc_t drs = make_rsrc(e.delta, (unsigned)e.sH * (unsigned)e.sW * 3u * (unsigned)sizeof(T));
    constexpr int TPS = kSegPixels / BM;
    const int MT = edge_segments(e) * TPS;
    for (int tile = blockIdx.x; tile < MT; tile += (int)nblk) {
        const int seg = tile / TPS, first = (tile - seg * TPS) * BM;
        __syncthreads();
        const int tot = tile_prologue(e, seg, first, BM, false, false, s_base, s_wy, s_wx, s_vm, sh);
        if (first >= tot) continue;                         // block-uniform
        if (first + wave * 32 >= tot) continue;             // no entry for this wave (no barrier until the next tile)
        const int pl = wave * 32 + p32;
        const bool act = first + pl < tot;
        const unsigned vmask = act ? s_vm[pl] : 0u;
        const int base3 = act ? s_base[pl] * 3 : 0;         // elements; negative for a border entry's first taps
        float in[KH];
#pragma unroll
        for (int st = 0; st < KH; ++st) {
            const int k0 = st, k1 = KH + st;                // the two halves of the wave
            const int off = h ? (k1 / 9) * 3 * e.sW + k1 % 9 : (k0 / 9) * 3 * e.sW + k0 % 9;
            const bool v = h ? (k1 < 27 && ((vmask >> (k1 < 27 ? k1 / 3 : 0)) & 1u)) : ((vmask >> (k0 / 3)) & 1u);
            const int byte = v ? (base3 + off) * (int)sizeof(T) : (int)0x80000000u;
            if constexpr (sizeof(T) == 2)
                in[st] = (float)__builtin_bit_cast(f16, __builtin_amdgcn_raw_buffer_load_b16(drs, byte, 0, 0));
            else
                in[st] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(drs, byte, 0, 0));
        }
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
        const float* wl = sW + h * KH * 32 + p32;
#pragma unroll
        for (int st = 0; st < KH; ++st) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wl[st * 32], in[st], acc, 0, 0, 0);
        // register r of a lane: cout 8 * (r / 4) + 4 * (lane / 32) + r % 4 of the tile, entry lane % 32
        if (act) {
            T* pp = (T*)e.P + pdst_offset(e, s_wy[pl], s_wx[pl]) + nt * 32 + 4 * h;
            if constexpr (sizeof(T) == 2) {
                f16x4 o[4];
#pragma unroll
                for (int g = 0; g < 4; ++g) o[g] = *reinterpret_cast<const f16x4*>(pp + 8 * g);
#pragma unroll
                for (int g = 0; g < 4; ++g) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) o[g][q] = (f16)((float)o[g][q] + acc[4 * g + q]);
                    *reinterpret_cast<f16x4*>(pp + 8 * g) = o[g];
                }
            } else {
                float4 o[4];
#pragma unroll
                for (int g = 0; g < 4; ++g) o[g] = *reinterpret_cast<const float4*>(pp + 8 * g);
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    o[g].x += acc[4 * g]; o[g].y += acc[4 * g + 1]; o[g].z += acc[4 * g + 2]; o[g].w += acc[4 * g + 3];
                    *reinterpret_cast<float4*>(pp + 8 * g) = o[g];
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Stem-type layers (few input channels, e.g. RGB): compile-time footprint
// KK x KK x CIN.  A thread owns one list entry and CPT couts; all of its
// KK*KK*CIN inputs are fetched up front (independent loads), the weights are
// broadcast from LDS ([tap][cin][cout], fp32).
// ---------------------------------------------------------------------------
template <typename T, int KK, int CIN, int CPT>
__global__ __launch_bounds__(256) void k_conv_small(EdgeBatch eb, int groups, int ppb) {
    const EdgeDev& e = eb.d[blockIdx.z];                  // blockIdx.z: stream of the batch
    extern __shared__ __align__(16) unsigned char smem[];
    float* sW = reinterpret_cast<float*>(smem);             // [tap][CIN][Cout]
    __shared__ int s_base[256], s_wy[256], s_wx[256];
    __shared__ unsigned s_vm[256];
    __shared__ int sh[8];
    constexpr int TAPS = KK * KK;
    const int tid = threadIdx.x;
    const int cg = tid % groups, pl = tid / groups;
    const T* __restrict__ delta = (const T*)e.delta;
    const T* __restrict__ w = (const T*)e.w;
    const int cc = CIN * e.Cout;
    carry_source_compaction(e, sh);
    for (int i = tid; i < TAPS * cc; i += 256) {
        const int tap = i / cc, r = i - tap * cc;
        const int co = r / CIN, ci = r - co * CIN;
        sW[tap * cc + ci * e.Cout + co] = (float)w[i];
    }
    long long block_taps = 0;
    const int tps = (kSegPixels + ppb - 1) / ppb;
    const int MT = edge_segments(e) * tps;
    for (int tile = blockIdx.x; tile < MT; tile += gridDim.x) {
        const int seg = tile / tps, first = (tile - seg * tps) * ppb;
        __syncthreads();
        const int tot = tile_prologue(e, seg, first, ppb, first == 0 && !e.up, true, s_base, s_wy, s_wx, s_vm, sh);
        if (first >= tot) continue;
        if (tid == 0) block_taps += sh[4];
        if (pl >= ppb || first + pl >= tot) continue;
        const unsigned vmask = s_vm[pl];
        const int base = s_base[pl];
        float in[TAPS * CIN];
#pragma unroll
        for (int tap = 0; tap < TAPS; ++tap) {
            const bool v = (vmask >> tap) & 1u;
            const T* src = delta + (v ? (size_t)(base + (tap / KK) * e.sW + (tap % KK)) * CIN : (size_t)0);
#pragma unroll
            for (int ci = 0; ci < CIN; ++ci) in[tap * CIN + ci] = (float)src[ci];
        }
#pragma unroll
        for (int tap = 0; tap < TAPS; ++tap)
            if (!((vmask >> tap) & 1u))
#pragma unroll
                for (int ci = 0; ci < CIN; ++ci) in[tap * CIN + ci] = 0.f;
        // the pending values this thread adds to travel while it multiplies (no upsampling: one pixel)
        const int f = 1 << e.up;
        T* pp0 = (T*)e.P + pdst_offset(e, s_wy[pl], s_wx[pl]) + cg * CPT;
        typename Row8<T>::reg pold[CPT / 8];
        if (f == 1) {
#pragma unroll
            for (int q = 0; q < CPT; q += 8) pold[q / 8] = Row8<T>::load(pp0 + q);
        }
        float acc[CPT];
#pragma unroll
        for (int q = 0; q < CPT; ++q) acc[q] = 0.f;
#pragma unroll
        for (int t = 0; t < TAPS * CIN; ++t) {
            const float a = in[t];
            const float* wt = sW + t * e.Cout + cg * CPT;
#pragma unroll
            for (int q = 0; q < CPT; q += 4) {
                const float4 w4 = *reinterpret_cast<const float4*>(wt + q);
                acc[q] = fmaf(a, w4.x, acc[q]); acc[q + 1] = fmaf(a, w4.y, acc[q + 1]);
                acc[q + 2] = fmaf(a, w4.z, acc[q + 2]); acc[q + 3] = fmaf(a, w4.w, acc[q + 3]);
            }
        }
        if (f == 1) {
#pragma unroll
            for (int q = 0; q < CPT; q += 8) Row8<T>::add_store(pp0 + q, pold[q / 8], acc + q);
            continue;
        }
        for (int ua = 0; ua < f; ++ua)
            for (int ub = 0; ub < f; ++ub) {
                T* pp = (T*)e.P + pdst_offset(e, s_wy[pl] + ua, s_wx[pl] + ub) + cg * CPT;
#pragma unroll
                for (int q = 0; q < CPT; q += 8) Row8<T>::add(pp + q, acc + q);
            }
    }
    if (tid == 0) add_macs(e, block_taps, 1);
}

// ---------------------------------------------------------------------------
// Plain FMA convolution for any dtype / channel count.
// Block = 16 list entries x 16 cout lanes; each thread keeps 4 couts at a time.
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void k_conv_plain(EdgeBatch eb) {
    const EdgeDev& e = eb.d[blockIdx.z];                  // blockIdx.z: stream of the batch
    __shared__ int s_base[16], s_wy[16], s_wx[16];
    __shared__ unsigned s_vm[16];
    __shared__ int sh[8];
    const int p = threadIdx.x >> 4, cl = threadIdx.x & 15;
    const T* __restrict__ delta = (const T*)e.delta;
    const T* __restrict__ w = (const T*)e.w;
    const int taps = e.k * e.k;
    constexpr int TPS = kSegPixels / 16;
    const int MT = edge_segments(e) * TPS;
    carry_source_compaction(e, sh);
    for (int tile = blockIdx.x; tile < MT; tile += gridDim.x) {
        const int seg = tile / TPS, first = (tile - seg * TPS) * 16;
        __syncthreads();
        const int tot = tile_prologue(e, seg, first, 16, first == 0 && !e.up, true, s_base, s_wy, s_wx, s_vm, sh);
        if (first >= tot) continue;
        if (threadIdx.x == 0) add_macs(e, sh[4], 1);
        if (first + p >= tot) continue;
        const unsigned vmask = s_vm[p];
        const int base = s_base[p], wy = s_wy[p], wx = s_wx[p];
        for (int cg = 0; cg < e.Cout; cg += 64) {
            float acc[4] = {0.f, 0.f, 0.f, 0.f};
            for (int tap = 0; tap < taps; ++tap) {
                if (!((vmask >> tap) & 1u)) continue;
                const int jy = tap / e.k, jx = tap - jy * e.k;
                const T* drow = delta + ((size_t)(base + jy * e.sW + jx)) * e.Cin;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int co = cg + cl + 16 * j;
                    if (co >= e.Cout) continue;
                    const T* wrow = w + ((size_t)(tap * e.Cout + co)) * e.Cin;
                    float a = acc[j];
                    for (int ci = 0; ci < e.Cin; ++ci) a = fmaf((float)drow[ci], (float)wrow[ci], a);
                    acc[j] = a;
                }
            }
            const int f = 1 << e.up;
            for (int ua = 0; ua < f; ++ua)
                for (int ub = 0; ub < f; ++ub) {
                    T* pp = (T*)e.P + pdst_offset(e, wy + ua, wx + ub);
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int co = cg + cl + 16 * j;
                        if (co < e.Cout) pp[co] = (T)((float)pp[co] + acc[j]);
                    }
                }
        }
    }
}

// Residual skip: P_dst[q] += delta[q] for every updated pixel q of the source.  A thread takes VEC channels of a pixel, nothing
// is ranked: the lists, marks and counts are left to the last npub blocks.  (Compacting a list segment first, a block to a
// segment and group of channels, took 7.2 to 8.0 us on the sites of a ResNet-18-style network of 296 x 424 frames, this 2.9 to 3.9.)
template <typename T, int VEC>
__global__ __launch_bounds__(256) void k_identity(unsigned npub, unsigned blocks, EdgeBatch eb) {
    EdgeDev e = eb.d[blockIdx.z];                         // blockIdx.z: stream of the batch
    const unsigned nblk = blocks - npub;
    if (blockIdx.x >= nblk) {
        publish_edge(e, blockIdx.x - nblk, npub);
        return;
    }
    read_now(e.delta, e.sflags, e.sH, e.sW, e.Cin, e.P, e.Cout, e.Hp, e.Wp, e.by0, e.bx0, e.p_oy, e.p_ox);
    const int chunks = e.Cin / VEC;
    const float rc = rcp_of(chunks), rw = rcp_of(e.sW);
    // (256 pieces at a time; 2^24 pixels of 4096 channels are more than 32 bits count)
    const long long total = (long long)e.sH * e.sW * chunks;
    for (long long i0 = (long long)blockIdx.x * 256; i0 < total; i0 += (long long)nblk * 256) {
        const int pix0 = (int)(i0 / chunks), r = (int)(i0 - (long long)pix0 * chunks) + (int)threadIdx.x;
        const int dp = div24(r, chunks, rc), pix = pix0 + dp, c0 = (r - dp * chunks) * VEC;
        if (i0 + threadIdx.x >= total || !(e.sflags[pix] & kFlagM)) continue;
        const int y = div24(pix, e.sW, rw), x = pix - y * e.sW;
        T* pp = (T*)e.P + pdst_offset(e, y + e.by0, x + e.bx0) + c0;
        const T* d = (const T*)e.delta + (size_t)pix * e.Cin + c0;
        if constexpr (VEC == 8) {
            f16x8 o = *reinterpret_cast<f16x8*>(pp);
            const f16x8 v = *reinterpret_cast<const f16x8*>(d);
#pragma unroll
            for (int q = 0; q < 8; ++q) o[q] = (f16)((float)o[q] + (float)v[q]);
            *reinterpret_cast<f16x8*>(pp) = o;
        } else {
#pragma unroll
            for (int q = 0; q < VEC; ++q) pp[q] = (T)((float)pp[q] + (float)d[q]);
        }
    }
}
template <typename T, int VEC>
static void launch_identity(const EdgeBatch& eb, int nb, hipStream_t st) {
    const EdgeDev& e = eb.d[0];
    const unsigned npub = publish_blocks(e), blocks = cap_blocks(((long long)e.sH * e.sW * (e.Cin / VEC) + 255) / 256, 65536) + npub;
    k_identity<T, VEC><<<dim3(blocks, 1, nb), dim3(256), 0, st>>>(npub, blocks, eb);
}

// Max pooling in delta form: for every destination view pixel whose window holds an
// updated source pixel, y = max of the source's activations f(A) over the in-view
// pixels of the window; P_dst += y - (newly unveiled ? 0 : previous output); the
// previous output is replaced by y.
template <typename T, int VEC> struct PoolVec {
    static __device__ __forceinline__ void load(const T* p, float* v) {
#pragma unroll
        for (int q = 0; q < VEC; ++q) v[q] = (float)p[q];
    }
    static __device__ __forceinline__ void store(T* p, const float* v) {
#pragma unroll
        for (int q = 0; q < VEC; ++q) p[q] = (T)v[q];
    }
};
template <> struct PoolVec<f16, 8> {
    static __device__ __forceinline__ void load(const f16* p, float* v) {
        const f16x8 t = *reinterpret_cast<const f16x8*>(p);
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = (float)t[q];
    }
    static __device__ __forceinline__ void store(f16* p, const float* v) {
        f16x8 t;
#pragma unroll
        for (int q = 0; q < 8; ++q) t[q] = (f16)v[q];
        *reinterpret_cast<f16x8*>(p) = t;
    }
};
template <> struct PoolVec<float, 4> {
    static __device__ __forceinline__ void load(const float* p, float* v) {
        const float4 t = *reinterpret_cast<const float4*>(p);
        v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    }
    static __device__ __forceinline__ void store(float* p, const float* v) {
        *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
    }
};

// Blocks per (list segment, group of kPoolChunks chunks of VEC channels): as many as the group has chunks, each takes its
// share of the segment's entries.  Neighbouring threads hold neighbouring chunks of an entry, so rows are read in whole
// lines: with a chunk per block, 16 bytes of every row, the boxes of a 720 x 1280 frame (64 channels) took 37 us, this 12.
// What bounds it: the way of the rows through the caches, each is read for up to four outputs.  KS: the window at compile
// time, whose rows then travel together, or 0.
constexpr int kPoolChunks = 8;
template <typename T, int VEC, int KS>
__global__ __launch_bounds__(256) void k_pool(EdgeBatch eb) {
    const EdgeDev& e = eb.d[blockIdx.z];                  // blockIdx.z: stream of the batch
    __shared__ int s_base[kSegPixels], s_wy[kSegPixels], s_wx[kSegPixels];
    __shared__ unsigned s_vm[kSegPixels];
    __shared__ int sh[8];
    const int nseg = edge_segments(e), k = KS ? KS : e.k;
    const int chunks = e.Cin / VEC, parts = chunks < kPoolChunks ? chunks : kPoolChunks;
    const int group = blockIdx.y / parts, part = blockIdx.y - group * parts;
    const int ch0 = group * kPoolChunks, nch = chunks - ch0 < kPoolChunks ? chunks - ch0 : kPoolChunks;
    const int share = (kSegPixels + parts - 1) / parts;   // entries of a block
    carry_source_compaction(e, sh);
    for (int seg = blockIdx.x; seg < nseg; seg += gridDim.x) {
        __syncthreads();
        // the destination's flags still hold this frame's N (set by the shift); marking the
        // pixels touched only ORs U in, so the channel chunks may read N at any time
        const int tot = tile_prologue(e, seg, 0, kSegPixels, blockIdx.y == 0, blockIdx.y == 0, s_base, s_wy, s_wx, s_vm, sh);
        const int first = part * share, n = tot - first < share ? tot - first : share;
        for (int i = threadIdx.x; i < n * nch; i += 256) {
            const int ent = first + i / nch, c0 = (ch0 + i % nch) * VEC;
            const int oy = s_wy[ent] - e.by0, ox = s_wx[ent] - e.bx0;          // view pixel of the destination
            // op == 2: the reset of a pixel zeroed its previous output as well (sites with crops, where a
            // reset pixel may be pooled in a later frame than the reset)
            const bool fresh = e.op == 1 && (e.dflags[oy * e.dW + ox] & kFlagN);
            const int yy = wrapc(e.d_aoy + oy, e.dH), yx = wrapc(e.d_aox + ox, e.dW);
            T* prev = (T*)e.dY + ((size_t)yy * e.dW + yx) * e.Cout + c0;
            T* pp = (T*)e.P + pdst_offset(e, s_wy[ent], s_wx[ent]) + c0;
            float pv[VEC], pd[VEC], y[VEC];
            PoolVec<T, VEC>::load(prev, pv);
            PoolVec<T, VEC>::load(pp, pd);
#pragma unroll
            for (int q = 0; q < VEC; ++q) y[q] = -INFINITY;
            auto tap = [&](int jy, int jx) {              // a tap outside the view reads one inside it and changes nothing
                const int iy = oy * e.stride - e.pad + jy, ix = ox * e.stride - e.pad + jx;
                const bool in = iy >= 0 && iy < e.sH && ix >= 0 && ix < e.sW;
                const int ay = wrapc(e.s_aoy + (in ? iy : 0), e.sH), ax = wrapc(e.s_aox + (in ? ix : 0), e.sW);
                float v[VEC];
                PoolVec<T, VEC>::load((const T*)e.sA + ((size_t)ay * e.sW + ax) * e.Cin + c0, v);
#pragma unroll
                for (int q = 0; q < VEC; ++q) {
                    const float m = fmaxf(y[q], e.s_relu ? fmaxf(v[q], 0.f) : v[q]);
                    y[q] = in ? m : y[q];
                }
            };
            if constexpr (KS > 0) {
#pragma unroll
                for (int t = 0; t < KS * KS; ++t) tap(t / KS, t % KS);
            } else {
                for (int jy = 0; jy < k; ++jy)
                    for (int jx = 0; jx < k; ++jx) tap(jy, jx);
            }
#pragma unroll
            for (int q = 0; q < VEC; ++q) pd[q] = (float)(T)(pd[q] + (y[q] - (fresh ? 0.f : pv[q])));
            PoolVec<T, VEC>::store(pp, pd);
            PoolVec<T, VEC>::store(prev, y);
        }
    }
}
template <typename T, int VEC>
static void launch_pool(const EdgeBatch& eb, int nb, unsigned segs, hipStream_t st) {
    const EdgeDev& e = eb.d[0];
    const int chunks = e.Cin / VEC, parts = chunks < kPoolChunks ? chunks : kPoolChunks;
    const dim3 grid(segs, (chunks + kPoolChunks - 1) / kPoolChunks * parts, nb);
    if (e.k == 3) k_pool<T, VEC, 3><<<grid, dim3(256), 0, st>>>(eb);
    else k_pool<T, VEC, 0><<<grid, dim3(256), 0, st>>>(eb);
}

// ---------------------------------------------------------------------------
// 1x1 convolution into a truncation-free site (no pending ring): for every destination pixel q
// whose source pixel was updated
//   t = round(y[q] (+ bias, if q is newly unveiled));  a = newly unveiled ? 0 : A[q]
//   A[q] <- a + t;  delta[q] <- f(a + t) - f(a);  updated if newly unveiled or any channel of the
//   delta is not zero
// which is what the pending ring and the delta kernel do with threshold 0.  A tile is a quarter of a
// list segment (64 destination pixels, the indices of one wave) and ALL output channels, so the block
// owns its pixels: it writes their flag bytes, also those of the pixels nobody touched - the mask of
// the frame is complete after this launch.  The first quarter also publishes the segment's compute list.
// fp16 with Cin % 16 == 0 and Cout % 32 == 0 runs on the matrix cores (operands straight from global
// memory: the layer is bound by the accumulated values it reads and writes); anything else takes one
// thread per (entry, output channel).
// ---------------------------------------------------------------------------
constexpr int kTfTile = 64;
template <typename T, bool MFMA>
__global__ __launch_bounds__(256) void k_conv_tf(EdgeBatch eb) {
    const EdgeDev& e = eb.d[blockIdx.z];                  // blockIdx.z: stream of the batch
    __shared__ int s_src[kTfTile], s_dst[kTfTile];
    __shared__ unsigned s_any[kTfTile];
    __shared__ uint8_t s_new[kTfTile];
    __shared__ int sh[8];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = e.dH * e.dW;                             // no border: the window is the view
    const int ntiles = ((n + kSegPixels - 1) / kSegPixels) * (kSegPixels / kTfTile);
    T* __restrict__ A = (T*)e.dY;
    T* __restrict__ D = (T*)const_cast<void*>(e.sA);
    const float* __restrict__ bias = (const float*)e.wp;
    const T* __restrict__ delta = (const T*)e.delta;
    const T* __restrict__ w = (const T*)e.w;
    carry_source_compaction(e, sh);
    long long block_taps = 0;                               // statistics (thread 0 only)
    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int seg = tile / (kSegPixels / kTfTile), quarter = tile % (kSegPixels / kTfTile);
        __syncthreads();                                    // previous tile is done with LDS
        const int p = seg * kSegPixels + tid;
        const bool own = wave == quarter;                   // this wave's 64 indices are the tile
        bool has = false;
        int fl = 0, src = 0;
        if (p < n) {
            const int oy = p / e.dW, ox = p - oy * e.dW;
            src = oy * e.stride * e.sW + ox * e.stride;       // k == 1, pad == 0: inside the source view
            has = (e.sflags[src] & kFlagM) != 0;
            if (own) fl = e.dflags[p];
        }
        if (tid < kTfTile) s_any[tid] = 0u;
        const unsigned long long bal = __ballot(has);
        const int rank = __popcll(bal & ((1ull << lane) - 1ull));
        if (lane == 0) sh[wave] = __popcll(bal);
        __syncthreads();
        const int tot = sh[quarter];
        if (own && has) {
            s_src[rank] = src;
            s_dst[rank] = p;
            s_new[rank] = (uint8_t)(fl & kFlagN);
        }
        if (quarter == 0) {                                // the segment's compute list, by its first tile
            int off = rank;
            for (int i = 0; i < wave; ++i) off += sh[i];
            if (has) e.clist[seg * kSegPixels + off] = p;
            if (tid == 0) {                                // single writer per segment: no atomics
                const int all = sh[0] + sh[1] + sh[2] + sh[3];
                e.ccnt[seg] = all;
                e.cacc[seg] += (unsigned long long)all;
            }
        }
        if (tid == 0) block_taps += tot;
        __syncthreads();
        if constexpr (MFMA) {
            // (32 entries x 32 couts) tiles dealt to the four waves; lane l feeds entry / cout l % 32 with
            // the 8 consecutive cin starting at 8 * (l / 32); register r of a lane holds cout
            // 8 * (r / 4) + 4 * (l / 32) + r % 4 of the tile for entry l % 32
            const int nra = (tot + 31) >> 5, nca = e.Cout >> 5;
            const int col = lane & 31, kh = lane >> 5;
            for (int u = wave; u < nra * nca; u += 4) {
                const int ra = u / nca, ca = u - ra * nca;
                const int ent = ra * 32 + col;
                const bool act = ent < tot;
                const f16* brow = (const f16*)delta + (size_t)s_src[act ? ent : 0] * e.Cin + kh * 8;
                const f16* arow = (const f16*)w + (size_t)(ca * 32 + col) * e.Cin + kh * 8;
                f32x16 acc;
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[r] = 0.f;
                int c0 = 0;
                for (; c0 + 64 <= e.Cin; c0 += 64) {           // four steps' operands are requested together
                    f16x8 a4[4], b4[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        a4[q] = *reinterpret_cast<const f16x8*>(arow + c0 + 16 * q);
                        b4[q] = *reinterpret_cast<const f16x8*>(brow + c0 + 16 * q);
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a4[q], b4[q], acc, 0, 0, 0);
                }
                for (; c0 < e.Cin; c0 += 16) {
                    const f16x8 a = *reinterpret_cast<const f16x8*>(arow + c0);
                    const f16x8 b = *reinterpret_cast<const f16x8*>(brow + c0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, acc, 0, 0, 0);
                }
                if (act) {                                   // (a dead column multiplied entry 0's row: dropped here)
                    const int p1 = s_dst[ent];
                    const int vy = p1 / e.dW, vx = p1 - vy * e.dW;
                    f16* Ap = (f16*)A + ((size_t)wrapc(e.d_aoy + vy, e.dH) * e.dW + wrapc(e.d_aox + vx, e.dW)) * e.Cout + ca * 32 + 4 * kh;
                    f16* Dp = (f16*)D + (size_t)p1 * e.Cout + ca * 32 + 4 * kh;
                    const bool fresh = s_new[ent] != 0;
                    f16x4 av[4];
#pragma unroll
                    for (int g = 0; g < 4; ++g) av[g] = *reinterpret_cast<const f16x4*>(Ap + 8 * g);
                    bool any = false;
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        f16x4 na, dv;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const float a = fresh ? 0.f : (float)av[g][i];
                            const float b = fresh && bias ? (float)(f16)bias[ca * 32 + 8 * g + 4 * kh + i] : 0.f;
                            const float t = (float)(f16)(b + acc[4 * g + i]);      // as the pending ring would hold it
                            const float sum = a + t;
                            const float out = e.s_relu ? fmaxf(sum, 0.f) - fmaxf(a, 0.f) : sum - a;
                            na[i] = (f16)sum;
                            dv[i] = (f16)out;
                            any |= out != 0.f;
                        }
                        *reinterpret_cast<f16x4*>(Ap + 8 * g) = na;
                        *reinterpret_cast<f16x4*>(Dp + 8 * g) = dv;
                    }
                    if (any) atomicOr(&s_any[ent], 1u);        // an OR: the order does not matter
                }
            }
        } else {
            for (int idx = tid; idx < tot * e.Cout; idx += 256) {
                const int ent = idx / e.Cout, co = idx - ent * e.Cout;
                const T* drow = delta + (size_t)s_src[ent] * e.Cin;
                const T* wrow = w + (size_t)co * e.Cin;
                float y = 0.f;
                for (int ci = 0; ci < e.Cin; ++ci) y = fmaf((float)drow[ci], (float)wrow[ci], y);
                const int p1 = s_dst[ent];
                const int vy = p1 / e.dW, vx = p1 - vy * e.dW;
                const size_t aoff = ((size_t)wrapc(e.d_aoy + vy, e.dH) * e.dW + wrapc(e.d_aox + vx, e.dW)) * e.Cout + co;
                const bool fresh = s_new[ent] != 0;
                const float a = fresh ? 0.f : (float)A[aoff];
                const float b = fresh && bias ? (float)(T)bias[co] : 0.f;
                const float t = (float)(T)(b + y);          // as the pending ring would hold it
                const float sum = a + t;
                const float out = e.s_relu ? fmaxf(sum, 0.f) - fmaxf(a, 0.f) : sum - a;
                A[aoff] = (T)sum;
                D[(size_t)p1 * e.Cout + co] = (T)out;
                if (out != 0.f) atomicOr(&s_any[ent], 1u);     // an OR: the order does not matter
            }
        }
        __syncthreads();
        if (own && p < n) e.dflags[p] = (uint8_t)(has ? ((((fl & kFlagN) || s_any[rank]) ? kFlagM : 0) | kFlagC) : 0);
    }
    if (tid == 0) add_macs(e, block_taps, MFMA ? 0 : 1);    // statistics: one atomic per block
}

// Compaction of the update mask alone (a forward call without outgoing edges).
__global__ __launch_bounds__(256) void k_compact_source(EdgeBatch eb) {
    const EdgeDev& e = eb.d[blockIdx.z];                  // blockIdx.z: stream of the batch
    __shared__ int sh[8];
    carry_source_compaction(e, sh);
}

// Tuning knobs (mdcnn_set_option): forced tile shape, pipeline depth, XCD mapping.
int g_tile = 0, g_pipe = 0, g_xcd = 1, g_kc = 0;
int g_f32_mfma = 1;     // 1: fp32 layers (k_conv_mfma_f32, k_conv_f32) and 3-channel stems go to the matrix cores where they apply, 0: plain FMA kernels

template <int WM, int WN, int TM, int TN, int KC, int PIPE>
static hipError_t launch_tiled(const EdgeBatch& eb, int nb, long long max_entries, hipStream_t st, ConvPick* pick, bool* read) {
    const EdgeDev& e = eb.d[0];
    using Cfg = TiledCfg<WM, WN, TM, TN, KC, PIPE>;
    const long long nseg = (max_entries + kSegPixels - 1) / kSegPixels;
    const long long MT = nseg * Cfg::TPS;
    const int NT = e.Cout / Cfg::BN;
    const int xcd = g_xcd && NT <= 8 && (8 % NT) == 0;
    const long long items = (xcd ? 8 * ((MT + 8 / NT - 1) / (8 / NT)) : MT * NT) * (e.up > 1 ? 1 << (2 * e.up - 2) : 1);
    unsigned g = cap_blocks(items, 4096);
    g = (g + 7u) & ~7u;                                    // whole rounds over the 8 XCDs
    const TileGrid tg{e.k == 1 || e.k == 3 ? publish_blocks(e) : 0u, e.up ? 0u : copy_blocks(e, 2), NT, xcd, 0, 0, 0u, 0u};
    g += tg.npub + tg.ncopy;
    if (read && tg.ncopy) *read = true;
    if (pick) {
        *pick = ConvPick{multi_tiled_body(WM, WN, TM, TN, KC, PIPE), (int)items, tg, g, (unsigned)Cfg::SMEM};
        return hipSuccess;
    }
    auto kern = k_conv_mfma_tiled<WM, WN, TM, TN, KC, PIPE>;
    // launches come from several host threads (frames in flight): the attribute is set once, by whoever is first
    static std::atomic<bool> attr_set{false};
    if (!attr_set.load(std::memory_order_acquire)) {
        hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, Cfg::SMEM);
        if (err != hipSuccess) { (void)hipGetLastError(); return err; }    // do not leave it for the next call to report
        attr_set.store(true, std::memory_order_release);
    }
    kern<<<dim3(g, 1, nb), dim3(256), Cfg::SMEM, st>>>(tg, g, (int)items, eb);
    return hipGetLastError();
}

template <int WM, int WN, int TM, int TN, int KC>
static hipError_t launch_tiled_p(const EdgeBatch& eb, int nb, long long max_entries, hipStream_t st, ConvPick* pick, bool* read) {
    const EdgeDev& e = eb.d[0];
    // measured on MI355X: with L2 latencies of ~200 cycles one step of prefetch is
    // enough; the second register stage only costs occupancy
    const bool deep = g_pipe == 2 && TiledCfg<WM, WN, TM, TN, KC, 2>::SMEM <= 150 * 1024;   // two stages must fit the LDS
    return deep ? launch_tiled<WM, WN, TM, TN, KC, 2>(eb, nb, max_entries, st, pick, read)
                : launch_tiled<WM, WN, TM, TN, KC, 1>(eb, nb, max_entries, st, pick, read);
}

// The largest tile that still yields about one block per compute unit.  A 1x1 edge that shares its launch leaves the
// places to the other one (two blocks to a compute unit, and a block more than that starts when the first are done:
// 3x3 and 1x1, 64 -> 128 channels on 130 x 130 pixels, 536 blocks 18.0 us, 403 blocks 16.0) - but takes 256 x 64, which the
// shared kernel does not carry, only where it fills the GPU by itself.
int gather_choice(long long entries, int k, int Cout, bool shared) {
    auto blocks = [&](int bm, int bn) { return (entries + bm - 1) / bm * (Cout / bn); };
    const long long want = shared && k == 1 ? 112 : 224;
    if (Cout % 128 == 0 && blocks(128, 128) >= want) return 4;
    if (Cout % 128 == 0 && blocks(64, 128) >= want) return 5;
    if (Cout % 64 == 0) return blocks(256, 64) >= 224 ? 1 : blocks(128, 64) >= want ? 2 : 3;
    return 6;
}
template <int KC>
static hipError_t launch_tiled_kc(const EdgeBatch& eb, int nb, long long max_entries, hipStream_t st, ConvPick* pick, bool* read) {
    const EdgeDev& e = eb.d[0];
    const int tile = g_tile ? g_tile : gather_choice(max_entries, e.k, e.Cout, pick != nullptr);
    switch (tile) {
        case 1: if (e.Cout % 64 == 0) return launch_tiled_p<4, 1, 2, 2, KC>(eb, nb, max_entries, st, pick, read); break;    // 256 x 64
        case 2: if (e.Cout % 64 == 0) return launch_tiled_p<2, 2, 2, 1, KC>(eb, nb, max_entries, st, pick, read); break;    // 128 x 64
        case 3: if (e.Cout % 64 == 0) return launch_tiled_p<2, 2, 1, 1, KC>(eb, nb, max_entries, st, pick, read); break;    //  64 x 64
        case 4: if (e.Cout % 128 == 0) return launch_tiled_p<2, 2, 2, 2, KC>(eb, nb, max_entries, st, pick, read); break;   // 128 x 128
        case 5: if (e.Cout % 128 == 0) return launch_tiled_p<2, 2, 1, 2, KC>(eb, nb, max_entries, st, pick, read); break;   //  64 x 128
        case 7: if (e.Cout % 128 == 0) return launch_tiled_p<4, 1, 1, 4, KC>(eb, nb, max_entries, st, pick, read); break;   // 128 x 128, wave 32 x 128
        case 8: if (e.Cout % 256 == 0) return launch_tiled_p<2, 2, 2, 4, KC>(eb, nb, max_entries, st, pick, read); break;   // 128 x 256, wave 64 x 128
        case 9: if (e.Cout % 256 == 0) return launch_tiled_p<1, 4, 2, 2, KC>(eb, nb, max_entries, st, pick, read); break;   //  64 x 256, wave 64 x 64
        case 10: if (e.Cout % 256 == 0) return launch_tiled_p<2, 2, 1, 4, KC>(eb, nb, max_entries, st, pick, read); break;  //  64 x 256, wave 32 x 128
        case 11: if (e.Cout % 128 == 0) return launch_tiled_p<1, 4, 1, 1, KC>(eb, nb, max_entries, st, pick, read); break;  //  32 x 128
        case 12: if (e.Cout % 256 == 0) return launch_tiled_p<1, 4, 1, 2, KC>(eb, nb, max_entries, st, pick, read); break;  //  32 x 256
        case 13: if (e.Cout % 128 == 0) return launch_tiled_p<1, 4, 2, 1, KC>(eb, nb, max_entries, st, pick, read); break;  //  64 x 128, wave 64 x 32
        case 14: if (e.Cout % 64 == 0) return launch_tiled_p<1, 4, 2, 1, 32>(eb, nb, max_entries, st, pick, read); break;   //  same, 32-channel steps
        default: break;
    }
    return launch_tiled_p<4, 1, 1, 1, KC>(eb, nb, max_entries, st, pick, read);                                             // 128 x 32
}

int g_halo = 1;          // 0: never use the halo-staged kernel, 2: force 32-cout tiles, 3: tiles are index ranges instead of
                         // rectangles (launch_halo_n), 4: as 1
int g_halo_sub = 0;      // 0: auto, 1 / 2 / 4: tiles per list segment of the halo-staged kernel

template <int NSUB, int WMV, int WK, int TM, int TN, int KC, int NLD, int RING = 3, int MINB = (NSUB >= 2 ? 2 : 1), bool T2D = false>
static hipError_t launch_halo_t(const EdgeBatch& eb, int nb, long long nseg, hipStream_t st, ConvPick* pick, int th = 0, int tw = 0) {
    const EdgeDev& e = eb.d[0];
    using Cfg = HaloCfg<NSUB, WMV, WK, TM, TN, KC, NLD, 3, RING, MINB>;
    const int NT = e.Cout / Cfg::BN;
    const long long tiles = T2D ? (long long)((e.Hp + th - 1) / th) * ((e.Wp + tw - 1) / tw) : nseg * NSUB;
    const long long items = tiles * NT;
    const unsigned npub = T2D ? publish_blocks(e) : 0u, blocks = cap_blocks(items, 16384) + npub;
    if (pick) {
        *pick = ConvPick{multi_halo_body(NSUB, WMV, WK, TM, TN, KC, NLD, RING, T2D), (int)items, TileGrid{npub, 0u, NT, th, tw, 0, 0u, 0u}, blocks, (unsigned)Cfg::SMEM};
        return hipSuccess;
    }
    auto kern = k_conv_halo<NSUB, WMV, WK, TM, TN, KC, NLD, 3, RING, MINB, T2D>;
    static std::atomic<bool> attr_set{false};
    if (!attr_set.load(std::memory_order_acquire)) {
        hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, Cfg::SMEM);
        if (err != hipSuccess) { (void)hipGetLastError(); return err; }    // do not leave it for the next call to report
        attr_set.store(true, std::memory_order_release);
    }
    kern<<<dim3(blocks, 1, nb), dim3(256), Cfg::SMEM, st>>>(eb, npub, NT, (int)items, th, tw);
    return hipGetLastError();
}

// Rectangle th x tw of at most `sub` pixels whose halo fits `cap` staged pixels, with the fewest tiles over an Hp x Wp window
// (ties: the smaller halo).  False if none fits.
static bool search_tile_2d(int Hp, int Wp, int k, int sub, int cap, int* th_out, int* tw_out, long long* tiles_out) {
    long long best = -1, best_halo = 0;
    for (int th = 1; th <= sub && th <= Hp; ++th) {
        int tw = sub / th < Wp ? sub / th : Wp;
        while (tw > 1 && (long long)(th + k - 1) * (tw + k - 1) > cap) --tw;
        if ((long long)(th + k - 1) * (tw + k - 1) > cap) continue;
        // the narrowest tile with the same number of columns of tiles
        const int cols = (Wp + tw - 1) / tw;
        tw = (Wp + cols - 1) / cols;
        const long long tiles = (long long)((Hp + th - 1) / th) * cols, halo = (long long)(th + k - 1) * (tw + k - 1);
        if (best < 0 || tiles < best || (tiles == best && halo < best_halo)) { best = tiles; best_halo = halo; *th_out = th; *tw_out = tw; }
    }
    if (best < 0) return false;
    *tiles_out = best;
    return true;
}
// The search takes some microseconds and every launch asks up to three times: the answers are kept per host thread, a few
// hundred at most (a network has a handful of window sizes).
bool tile_2d(int Hp, int Wp, int k, int sub, int cap, int* th_out, int* tw_out, long long* tiles_out) {
    struct Entry { int Hp = -1, Wp, k, sub, cap, th, tw; bool fits; long long tiles; };
    static thread_local Entry table[256];
    const unsigned h = (unsigned)Hp * 2654435761u ^ (unsigned)Wp * 2246822519u ^ (unsigned)(sub * 8 + k) * 3266489917u ^ (unsigned)cap * 668265263u;
    Entry& t = table[(h >> 16) % 256];
    if (t.Hp != Hp || t.Wp != Wp || t.k != k || t.sub != sub || t.cap != cap) {
        t = Entry{Hp, Wp, k, sub, cap, 0, 0, false, 0};
        t.fits = search_tile_2d(Hp, Wp, k, sub, cap, &t.th, &t.tw, &t.tiles);
    }
    if (!t.fits) return false;
    *th_out = t.th;
    *tw_out = t.tw;
    *tiles_out = t.tiles;
    return true;
}

// Rectangle of at most m pixels for the tiles of conv_rect.h, whose footprint fits `rows` rows of 16, with the fewest tiles over
// an Hp x Wp window (ties: the smaller footprint).  Asked for by every launch: the answers are kept per host thread, as tile_2d's.
void rect_tile(int Hp, int Wp, int m, int rows, int stride, int* th_out, int* tw_out, long long* tiles_out) {
    struct Entry { int Hp = -1, Wp, m, rows, stride, th, tw; long long tiles; };
    static thread_local Entry table[256];
    const unsigned h = (unsigned)Hp * 2654435761u ^ (unsigned)Wp * 2246822519u ^ (unsigned)(m * 64 + rows * 2 + stride) * 3266489917u;
    Entry& t = table[(h >> 16) % 256];
    if (t.Hp != Hp || t.Wp != Wp || t.m != m || t.rows != rows || t.stride != stride) {
        t = Entry{Hp, Wp, m, rows, stride, 0, 0, -1};
        long long halo = 0;
        const int highest = (rows - 3) / stride + 1, widest = 13 / stride + 1;
        for (int tw = 1; tw <= widest && tw <= Wp; ++tw) {
            int th = m / tw < highest ? m / tw : highest;
            if (th > Hp) th = Hp;
            const int down = (Hp + th - 1) / th, across = (Wp + tw - 1) / tw;
            th = (Hp + down - 1) / down;                   // the lowest tile with as many rows of tiles
            const long long n = (long long)down * across, hl = (long long)((th - 1) * stride + 3) * ((tw - 1) * stride + 3);
            if (t.tiles < 0 || n < t.tiles || (n == t.tiles && hl < halo)) { t.tiles = n; halo = hl; t.th = th; t.tw = tw; }
        }
    }
    *th_out = t.th;
    *tw_out = t.tw;
    *tiles_out = t.tiles;
}
template <typename Cfg>
static hipError_t launch_rect_t(const EdgeBatch& eb, int nb, hipStream_t st, ConvPick* pick, bool* done, bool* read) {
    const EdgeDev& e = eb.d[0];
    int th, tw;
    long long tiles;
    static_assert(Cfg::S != 1 || Cfg::ROWS == rect_rows(Cfg::M), "the rows mdcnn_rect_tiles counts on");
    rect_tile(e.Hp, e.Wp, Cfg::M, Cfg::ROWS, Cfg::S, &th, &tw, &tiles);
    const int NT = e.Cout / Cfg::BN, tiles_x = (e.Wp + tw - 1) / tw;
    *done = (double)tiles * NT * NT < 4e9 && (double)tiles * tiles_x < 4e9;      // (the reciprocals are exact below 2^32)
    if (!*done) return hipSuccess;
    const unsigned npub = publish_blocks(e), ncopy = copy_blocks(e, 2), blocks = (unsigned)(tiles * NT) + npub + ncopy;
    if (read && ncopy) *read = true;
    const TileGrid g{npub, ncopy, NT, th, tw, tiles_x, reciprocal_of((unsigned)NT), reciprocal_of((unsigned)tiles_x)};
    if (pick) {
        *pick = ConvPick{rect_body_number<Cfg>(), (int)(tiles * NT), g, blocks, (unsigned)Cfg::SMEM};
        return hipSuccess;
    }
    auto kern = k_conv_rect<Cfg>;
    static std::atomic<bool> attr_set{false};
    if (!attr_set.load(std::memory_order_acquire)) {
        hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, Cfg::SMEM);
        if (err != hipSuccess) { (void)hipGetLastError(); return err; }    // do not leave it for the next call to report
        attr_set.store(true, std::memory_order_release);
    }
    kern<<<dim3(blocks, 1, nb), dim3(256), Cfg::SMEM, st>>>(g, blocks, eb);
    return hipGetLastError();
}

// Which tile: entries (*m) and couts / 32 (*tn).
// Couts: a launch of few tiles takes 32 to a tile instead of 64: half the products and weights to a tile, twice the tiles (the
// low resolutions of the HRNet-like network, 20 to 40 tiles: frame 496 -> 480 us; 0 to 128 in place of 64 for frames in flight: no
// difference).  No sum changes with it.
// Entries.  Alone on the GPU a launch takes as long as the compute unit with the most tiles, one or two of them, and a tile
// as long as its K loop (per entry, Cin + what the epilogue takes); with several tiles per compute unit it is the sum of the
// tiles and 2 us of each (12500 in these units) that nothing
// covers.  Tiles of 160 entries have a compute unit for themselves and an epilogue that takes 1.3 us more; nothing covers
// theirs, so they are for launches that are not full (a ResNet-18-style batch frame by frame, 512 x 512, with / without this: 4
// videos 3951 / 3730 frames/s, 8 videos 4480 / 4080, 16 videos 4750 / 4310).  Measured alone, 64 /
// 96 / 160 entries: 512 -> 512 channels on a 66 x 66 window 30.9 / 25.2 / 23.2 us (29.9 with the kernel before), 256 -> 256
// 12.5 / 10.6 / 15.2 (13.3), 128 -> 128 on 130 x 130 14.2 / 11.2 / 12.3 (12.8); 16 videos, 96 / 128 / 160 entries: 293 / 264
// / 308 us (279), 84 / 78 / 100 (81), 95 / 91 / 129 (96).  64 channels on large windows: 256-entry tiles without a K split,
// two to a compute unit, 12.4 us on 258 x 258 against 17.7 with 160-entry tiles, 16 videos 111 (13.6 and 118 before).
// Frames in flight: about three launches share the 512 places, so a launch has some 170.  With fewer tiles it takes as long as
// one tile, with more as their sum divided by its places; equal cost, the smaller tile.  (Clips of 30 frames, this rule / four times
// the tiles and a step at two per compute unit / 64 / 96 / 128 entries everywhere: 256 x 256 3848 / 3975 / 3850 / 3966 / 4349
// us, 288 x 288 4120 / 4453 / 4159 / 4121 / 4459, 320 x 320 4363 / 4630 / 4469 / 4398 / 4618, 512 x 512 7047 / 7034 / 7648 / 7151
// / 7043, 640 x 640 9870 / 9843 / - / 10055 / -.)  A tile costs the row tiles it has, not those it could have (18 x 18 windows
// are four of 81 pixels, three row tiles, under the limit of 128), and its weights, as much as 16 entries' products: batches
// of 8 in flight, pooling stem, 512 x 512, 12.8 -> 13.1 k frames/s, 16 videos of 256 x 256 4.72 -> 4.51 ms.
void rect_choice(int Hp, int Wp, int Cin, int Cout, int nb, bool alone, bool shared, int* tn, int* m_out) {
    auto tiles_of = [&](int m, int couts, int* pixels = nullptr) {
        int th, tw;
        long long tiles;
        rect_tile(Hp, Wp, m, rect_rows(m), 1, &th, &tw, &tiles);
        if (pixels) *pixels = (th * tw + 31) / 32 * 32;
        return tiles * (Cout / couts);
    };
    *tn = Cout % 64 == 0 && g_halo != 2 && (g_halo_sub || tiles_of(64, 64) * nb > 64) ? 2 : 1;
    if (g_halo_sub) {
        *m_out = g_halo_sub == 4 ? 64 : g_halo_sub == 2 ? 128 : Cin == 64 ? 256 : 160;
        return;
    }
    if (Cin == 64 && tiles_of(96, 32 * *tn) > 512) {
        *m_out = 256;
        return;
    }
    double best = 0;
    *m_out = 0;
    for (int px = 64; px <= (alone && !shared ? 160 : 128); px += 32) {
        int pixels;                                        // (a K loop walks the 32-pixel row tiles that a tile has)
        const double tiles = (double)(tiles_of(px, 32 * *tn, &pixels) * nb), loop = (double)(alone ? px : pixels) * (Cin + 78);
        double cost;
        if (alone) {
            const double per_cu = tiles / 256;
            if (per_cu > 2 && px == 160) continue;
            cost = (per_cu > 2 ? per_cu : per_cu <= 1 ? 1 : 2) * (loop + (per_cu > 2 ? 12500 : px == 160 ? 8000 : 0));
        } else {
            const double turns = tiles * 3 / 512;
            cost = (turns > 1 ? turns : 1) * (loop + 16 * Cin + 12500);
        }
        if (shared && tiles > 352) cost *= 1.4;            // beside the blocks of other edges: some would wait for a place
        if (*m_out == 0 || (alone ? cost <= best : cost < best)) { best = cost; *m_out = px; }
    }
}
template <int TN>
static hipError_t launch_rect(const EdgeBatch& eb, int nb, int m, hipStream_t st, ConvPick* pick, bool* done, bool* read) {
    using T = RectTiles<TN>;
    switch (m) {
        case 64: return launch_rect_t<typename T::T64>(eb, nb, st, pick, done, read);
        case 96: return launch_rect_t<typename T::T96>(eb, nb, st, pick, done, read);
        case 128: return launch_rect_t<typename T::T128>(eb, nb, st, pick, done, read);
        case 160: return launch_rect_t<typename T::T160>(eb, nb, st, pick, done, read);
        default: return launch_rect_t<typename T::T256>(eb, nb, st, pick, done, read);
    }
}

// Stride 2: tiles of 64 entries (at most 7 columns: the footprint of 15 columns is a row of 16 staged pixels), couts / 32 by the
// number of tiles: 32 couts where a launch has few (rect_choice), 128 where 64 would take more than a compute unit's share of
// blocks twice - a tile is round trips whatever it multiplies, and its footprint is staged once for 128 couts.  64 -> 128
// channels on 129 x 129 pixels beside the projection of the block: 64 couts 18.0 us, 128 couts 13.1, the gather tiles before
// 15.1; 128 -> 256 on 65 x 65: 15.7, 12.7, 14.6; 16 videos of them 99 / 87 / 85 and 101 / 76 / 79.  64 -> 64 on 97 x 73
// 8.1 us (gather tiles 12.1), 32 -> 32 on 49 x 37 5.5 (11.4): HRNet-like 384 x 288 frame 471 -> 439 us.
// The one batch that the gather tiles are ahead in does not go to them: they add up in another order, and a video of a batch gives
// the bits it gives alone.  Nor does a scene that stands still, of which nobody knows beforehand: the launch of 16 HRNet-like 512 x 512
// videos, 64 -> 64, takes 30 us for 15 when there is nothing to do.  Weights and rows asked for once a tile is known to have entries took
// 6 us off such a frame of 1101 and added 6 to the frame of 8 videos of 972, in the launches that carry these tiles beside others.
int rect_choice_s2(int Hp, int Wp, int Cin, int Cout, int nb) {
    int th, tw;
    long long tiles;
    rect_tile(Hp, Wp, 64, 16, 2, &th, &tw, &tiles);
    tiles = tiles * nb * (Cout / 64);
    if (Cout % 64 || g_halo == 2 || tiles <= 64) return 1;
    return Cout % 128 || Cin % 64 || tiles <= 256 ? 2 : 4;
}
template <int TN>
static hipError_t launch_rect_s2(const EdgeBatch& eb, int nb, hipStream_t st, ConvPick* pick, bool* done, bool* read) {
    using T = RectTiles<TN>;
    const int Cin = eb.d[0].Cin;
    if (Cin == 64) return launch_rect_t<typename T::S2One>(eb, nb, st, pick, done, read);
    if (Cin % 64 == 0) return launch_rect_t<typename T::S2>(eb, nb, st, pick, done, read);
    if constexpr (TN <= 2) return launch_rect_t<typename T::S2Half>(eb, nb, st, pick, done, read);
    else return hipErrorInvalidValue;
}

// Rectangular tiles of the layers whose input channels are a multiple of 32 and not of 64.  The tile size follows the number
// of tiles of ONE stream, whatever the batch - the K split of a tile fixes the order of the sums, and a stream in a batch must
// give the bits it gives alone: whole segments if that gives every compute unit a tile, else the smallest split that gives
// half of them one.  A whole-segment tile keeps its four waves on rows (no K split: 64 accumulator registers, two tiles per
// compute unit).
template <int TN>
static hipError_t launch_halo_2d(const EdgeBatch& eb, int nb, hipStream_t st, ConvPick* pick, bool* done) {
    const EdgeDev& e = eb.d[0];
    const int NT = e.Cout / (32 * TN);
    int th = 0, tw = 0;
    long long tiles = 0;
    *done = e.Cin % 32 == 0;
    if (!*done) return hipSuccess;
    const int first = g_halo_sub ? g_halo_sub : 1;
    for (int nsub = first; nsub <= 4; nsub *= 2) {
        const int sub = kSegPixels / nsub;
        // whole segments if every compute unit gets a tile, else the smallest split that gives at least half of them one
        // (a forced split is taken as it is)
        if (!g_halo_sub && nsub < 4 && tile_2d(e.Hp, e.Wp, e.k, sub, 1 << 20, &th, &tw, &tiles) && tiles * NT < (nsub == 1 ? 256 : 128)) continue;
        if (nsub == 1) {
            if (tile_2d(e.Hp, e.Wp, e.k, sub, HaloCfg<1, 4, 1, 2, TN, 32, 6, 3>::CAP, &th, &tw, &tiles))
                return launch_halo_t<1, 4, 1, 2, TN, 32, 6, 3, 2, true>(eb, nb, 0, st, pick, th, tw);
        } else if (nsub == 2) {
            if (tile_2d(e.Hp, e.Wp, e.k, sub, HaloCfg<2, 2, 2, 2, TN, 32, 3, 3>::CAP, &th, &tw, &tiles))
                return launch_halo_t<2, 2, 2, 2, TN, 32, 3, 3, 2, true>(eb, nb, 0, st, pick, th, tw);
        } else if (tile_2d(e.Hp, e.Wp, e.k, sub, HaloCfg<4, 2, 2, 1, TN, 32, 2, 3>::CAP, &th, &tw, &tiles)) {
            return launch_halo_t<4, 2, 2, 1, TN, 32, 2, 9, 2, true>(eb, nb, 0, st, pick, th, tw);
        }
    }
    *done = false;
    return hipSuccess;
}

// Staged pixels the rectangle of `sub` consecutive window indices can need.
static long long halo_worst(const EdgeDev& e, int sub) {
    const long long span = (sub - 2) / e.Wp + 2;                            // window rows the range can straddle
    const long long width = span > 1 || sub > e.Wp ? e.Wp : sub;
    return (span + e.k - 1) * (width - 1 + e.k);
}

// Tiles that are index ranges of the padded window (MDCNN_OPT_CONV_HALO = 3 only: rectangles fit every window and are
// ahead; the tests compare the two bit for bit), where the rectangle of pixels a range can read fits the staging buffer
// (the fewer channels per chunk, the more pixels fit; below 32 channels per chunk
// -- rows wider than about 250 pixels -- the tiled kernel is faster).
// *done = false: not applicable.
// Tiles are whole segments, halves or quarters: the smallest split that keeps at
// least half of the compute units busy (measured: finer splits re-read the weights
// more often than the extra parallelism pays back).
template <int TN>
static hipError_t launch_halo_n(const EdgeBatch& eb, int nb, long long nseg, hipStream_t st, ConvPick* pick, bool* done) {
    const EdgeDev& e = eb.d[0];
    const long long per_split = nseg * (e.Cout / (32 * TN));
    int nsub = g_halo_sub ? g_halo_sub : (per_split >= 256 ? 1 : per_split * 2 >= 128 ? 2 : 4);
    *done = true;
    for (; nsub <= 4; nsub *= 2) {
        const long long worst = halo_worst(e, kSegPixels / nsub);
        const bool c64 = e.Cin % 64 == 0, c32 = e.Cin % 32 == 0;
        if (nsub == 1) {
            if (c64 && worst <= HaloCfg<1, 2, 2, 4, TN, 64, 16, 3>::CAP) return launch_halo_t<1, 2, 2, 4, TN, 64, 16>(eb, nb, nseg, st, pick);
            if (c32 && worst <= HaloCfg<1, 2, 2, 4, TN, 32, 12, 3>::CAP) return launch_halo_t<1, 2, 2, 4, TN, 32, 12>(eb, nb, nseg, st, pick);
        } else if (nsub == 2) {
            // (split four ways as the rectangles are; 32 couts whatever TN: with 64 the accumulators of four row tiles leave no registers)
            if (c64 && worst <= HaloCfg<2, 1, 4, 4, 1, 64, 11, 3>::CAP) return launch_halo_t<2, 1, 4, 4, 1, 64, 11>(eb, nb, nseg, st, pick);
            if (c32 && worst <= HaloCfg<2, 2, 2, 2, TN, 32, 9, 3>::CAP) return launch_halo_t<2, 2, 2, 2, TN, 32, 9>(eb, nb, nseg, st, pick);
        } else {
            if (c64 && worst <= HaloCfg<4, 1, 4, 2, TN, 64, 9, 3>::CAP) return launch_halo_t<4, 1, 4, 2, TN, 64, 9, 9>(eb, nb, nseg, st, pick);
            if (c32 && worst <= HaloCfg<4, 2, 2, 1, TN, 32, 6, 3>::CAP) return launch_halo_t<4, 2, 2, 1, TN, 32, 6, 9>(eb, nb, nseg, st, pick);
        }
    }
    *done = false;
    return hipSuccess;
}

static hipError_t launch_halo(const EdgeBatch& eb, int nb, long long nseg, bool alone, hipStream_t st, ConvPick* pick, bool* done, bool* read) {
    const EdgeDev& e = eb.d[0];
    *done = false;
    if (!g_halo || !e.wp || e.k != 3 || e.stride > 2 || e.up != 0 || e.Cin % 16 || e.Cout % 32) return hipSuccess;
    if ((long long)e.sH * e.sW * e.Cin >= (1ll << 30) || (long long)e.k * e.k * e.Cin * e.Cout >= (1ll << 30))
        return hipSuccess;                                                     // 32-bit byte offsets into deltas and weights
    if (e.stride == 2) {
        if (g_halo == 3 || e.Cin % 32) return hipSuccess;
        const int tn = rect_choice_s2(e.Hp, e.Wp, e.Cin, e.Cout, nb);
        return tn == 1 ? launch_rect_s2<1>(eb, nb, st, pick, done, read) : tn == 2 ? launch_rect_s2<2>(eb, nb, st, pick, done, read)
                                                                                  : launch_rect_s2<4>(eb, nb, st, pick, done, read);
    }
    // Rectangular tiles (one of up to 64 pixels fits every window).  Windows of a few list segments used to stay on index
    // ranges, whose tiles stage whole rows; with the by-products made by other blocks and the round trips of a small tile
    // overlapped the rectangles are faster there too: HRNet-like network 659 -> 611 us a frame, 37 x 53 windows of 256 and 512
    // channels 22 -> 17 us a launch.
    if (g_halo != 3 && e.Cin % 64 == 0) {
        int tn, m;
        rect_choice(e.Hp, e.Wp, e.Cin, e.Cout, nb, alone, pick != nullptr, &tn, &m);
        return tn == 2 ? launch_rect<2>(eb, nb, m, st, pick, done, read) : launch_rect<1>(eb, nb, m, st, pick, done, read);
    }
    if (g_halo != 3) return e.Cout % 64 == 0 && g_halo != 2 ? launch_halo_2d<2>(eb, nb, st, pick, done) : launch_halo_2d<1>(eb, nb, st, pick, done);
    return e.Cout % 64 == 0 ? launch_halo_n<2>(eb, nb, nseg, st, pick, done) : launch_halo_n<1>(eb, nb, nseg, st, pick, done);
}

hipError_t launch_pack_weights(const void* src, void* dst, int taps, int Cout, int Cin, hipStream_t st) {
    const long long n8 = (long long)taps * Cout * Cin / 8;
    k_pack_weights<<<dim3(cap_blocks((n8 + 255) / 256, 2048)), dim3(256), 0, st>>>((const f16*)src, (f16*)dst, taps, Cout, Cin);
    return hipGetLastError();
}

template <typename T>
static hipError_t launch_ldsw(const EdgeBatch& eb, int nb, long long max_entries, hipStream_t st) {
    const EdgeDev& e = eb.d[0];
    const int groups = e.Cout / 8, ppb = 256 / groups;
    const size_t smem = (size_t)e.k * e.k * e.Cin * e.Cout * 4;
    auto kern = k_conv_ldsw<T>;
    if (smem > 65536) {
        // the limit only grows; the lock keeps two host threads from lowering it under each other
        static std::mutex mu;
        static size_t attr_bytes = 0;
        std::lock_guard<std::mutex> lock(mu);
        if (smem > attr_bytes) {
            hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
            if (err != hipSuccess) return err;
            attr_bytes = smem;
        }
    }
    const long long nseg = (max_entries + kSegPixels - 1) / kSegPixels;
    const long long tps = (kSegPixels + ppb - 1) / ppb;
    // weights are staged once per block: keep the blocks few and persistent
    unsigned g = cap_blocks(nseg * tps, smem > 32768 ? 256 : 768);
    kern<<<dim3(g, 1, nb), dim3(256), smem, st>>>(eb, groups, ppb);
    return hipGetLastError();
}

// fp32 layers the matrix cores take (k_conv_mfma_f32); *done = false: not this layer
template <int KK, int CIN, int KS>
static hipError_t launch_mfma_f32_inst(const EdgeBatch& eb, int nb, long long nseg, hipStream_t st, bool* read) {
    const EdgeDev& e = eb.d[0];
    static std::atomic<bool> attr_set{false};
    auto kern = k_conv_mfma_f32<KK, CIN, KS>;
    const size_t smem = (size_t)KK * KK * CIN * 32 * 4;
    if (smem > 49152 && !attr_set.load(std::memory_order_acquire)) {
        hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (err != hipSuccess) return err;
        attr_set.store(true, std::memory_order_release);
    }
    const int nts = (e.Cout + 31) / 32;
    const long long tiles = nseg * (kSegPixels / (32 * (4 / KS)));
    // weights are staged once per block: a bounded number of persistent blocks
    const long long cap = (smem > 49152 ? 512 : 1024) / nts;
    const unsigned npub = publish_blocks(e), ncopy = copy_blocks(e, 4), g = cap_blocks(tiles, cap > 0 ? cap : 1) + npub + ncopy;
    if (read && ncopy) *read = true;
    kern<<<dim3(g, nts, nb), dim3(256), smem, st>>>(npub, ncopy, g, eb);
    return hipGetLastError();
}
template <int KK, int CIN>
static hipError_t launch_mfma_f32_ks(const EdgeBatch& eb, int nb, long long nseg, hipStream_t st, bool* read) {
    const EdgeDev& e = eb.d[0];
    if constexpr (KK == 1) {
        return launch_mfma_f32_inst<KK, CIN, 1>(eb, nb, nseg, st, read);
    } else {
        // two waves share the taps of a 64-entry tile unless 128-entry tiles already give every compute unit four
        // blocks (measured on 32- and 64-channel layers of 66 and 17 segments: 10.5 k frames/s of a small network with one wave
        // per tile, 11.7 k with two, 10.4 k with four)
        const long long nts = (e.Cout + 31) / 32;
        int ks = nseg * 2 * nts >= 1024 ? 1 : 2;
        if (g_tile == 1 || g_tile == 2 || g_tile == 4) ks = g_tile;
        if (ks == 1) return launch_mfma_f32_inst<KK, CIN, 1>(eb, nb, nseg, st, read);
        if (ks == 2) return launch_mfma_f32_inst<KK, CIN, 2>(eb, nb, nseg, st, read);
        return launch_mfma_f32_inst<KK, CIN, 4>(eb, nb, nseg, st, read);
    }
}
static hipError_t launch_mfma_f32(const EdgeBatch& eb, int nb, long long nseg, hipStream_t st, bool* done, bool* read) {
    const EdgeDev& e = eb.d[0];
    *done = false;
    if (e.up || (e.k != 1 && e.k != 3) || (e.Cin != 16 && (e.k == 3 || (e.Cin != 32 && e.Cin != 64))) || (e.Cout % 32 != 0 && e.Cout != 16) || e.Cout > 1024 ||
        (long long)e.sH * e.sW * e.Cin >= (1ll << 29) || (long long)e.k * e.k * e.Cin * e.Cout >= (1ll << 29))
        return hipSuccess;
    *done = true;
    if (e.k == 3) return launch_mfma_f32_ks<3, 16>(eb, nb, nseg, st, read);
    return e.Cin == 16 ? launch_mfma_f32_ks<1, 16>(eb, nb, nseg, st, read)
         : e.Cin == 32 ? launch_mfma_f32_ks<1, 32>(eb, nb, nseg, st, read) : launch_mfma_f32_ks<1, 64>(eb, nb, nseg, st, read);
}

// Upsampling 1x1 edges of 64 n channels; *done: false if the edge is not one of them.
static hipError_t launch_up(const EdgeBatch& eb, int nb, hipStream_t st, ConvPick* pick, bool* done, bool* read) {
    const EdgeDev& e = eb.d[0];
    const long long HW = (long long)e.sH * e.sW, MT = (HW + kUpPx - 1) / kUpPx, NT = e.Cout / kUpCo, tiles = MT * up_parts(e.up);
    *done = e.k == 1 && e.up && e.Cin % 64 == 0 && HW * e.Cin < (1ll << 30) && (long long)e.Cin * e.Cout < (1ll << 30) && (long long)e.dH * e.dW < (1ll << 31) &&
            (double)tiles * NT * NT < 4e9 && (double)tiles * MT < 4e9;        // (the reciprocals are exact below 2^32)
    if (!*done) return hipSuccess;
    const unsigned npub = publish_blocks(e), ncopy = copy_blocks(e, 2), blocks = (unsigned)(tiles * NT) + npub + ncopy;
    if (read && ncopy) *read = true;
    const int early = nb * HW * (e.Cin + ((long long)e.Cout << (2 * e.up))) <= 8 << 20;
    const TileGrid g{npub, ncopy, (int)NT, 0, 0, (int)MT, reciprocal_of((unsigned)NT), reciprocal_of((unsigned)MT), early};
    if (pick) {
        *pick = ConvPick{kMultiUpBody, 0, g, blocks, (unsigned)kUpSmem};
        return hipSuccess;
    }
    k_conv_up<<<dim3(blocks, 1, nb), dim3(256), kUpSmem, st>>>(g, blocks, eb);
    return hipGetLastError();
}

hipError_t launch_conv(const EdgeBatch& eb, int nb, int dtype, int conv_path, bool alone, hipStream_t st, int* cls, ConvPick* pick, bool* read) {
    const EdgeDev& e = eb.d[0];                            // geometry and weights layout are the same for all streams
    const long long max_entries = e.up ? (long long)e.sH * e.sW : (long long)e.Hp * e.Wp;
    const long long nseg = (max_entries + kSegPixels - 1) / kSegPixels;
    if (pick) pick->body = -1;
    if (pick && (e.k <= 0 || e.op)) return hipSuccess;
    if (e.k < 0) {                                         // no operator: source compaction only
        *cls = kClsLists;
        k_compact_source<<<dim3(cap_blocks(((long long)e.sH * e.sW + kSegPixels - 1) / kSegPixels, 4096), 1, nb), dim3(256), 0, st>>>(eb);
        return hipGetLastError();
    }
    if (e.op == kOpTruncFree) {
        const bool mfma = dtype == MDCNN_F16 && conv_path != 1 && e.Cin % 16 == 0 && e.Cout % 32 == 0;
        *cls = mfma ? kClsConvMfma : kClsConvPlain;
        const unsigned g = cap_blocks((((long long)e.dH * e.dW + kSegPixels - 1) / kSegPixels) * (kSegPixels / kTfTile), 8192);
        if (mfma) k_conv_tf<f16, true><<<dim3(g, 1, nb), dim3(256), 0, st>>>(eb);
        else if (dtype == MDCNN_F16) k_conv_tf<f16, false><<<dim3(g, 1, nb), dim3(256), 0, st>>>(eb);
        else k_conv_tf<float, false><<<dim3(g, 1, nb), dim3(256), 0, st>>>(eb);
        return hipGetLastError();
    }
    if (e.op) {
        *cls = kClsPool;
        const unsigned g = cap_blocks(nseg, 4096);
        if (dtype == MDCNN_F16) {
            if (e.Cin % 8 == 0) launch_pool<f16, 8>(eb, nb, g, st);
            else launch_pool<f16, 1>(eb, nb, g, st);
        } else {
            if (e.Cin % 4 == 0) launch_pool<float, 4>(eb, nb, g, st);
            else launch_pool<float, 1>(eb, nb, g, st);
        }
        return hipGetLastError();
    }
    if (e.k == 0) {
        *cls = kClsIdentity;
        if (dtype == MDCNN_F16) {
            if (e.Cin % 8 == 0) launch_identity<f16, 8>(eb, nb, st);
            else launch_identity<f16, 1>(eb, nb, st);
        } else {
            if (e.Cin % 4 == 0) launch_identity<float, 4>(eb, nb, st);
            else launch_identity<float, 1>(eb, nb, st);
        }
        return hipGetLastError();
    }
    // conv_path: 0 auto, 1 plain FMA (per-thread weights), 2 MFMA without LDS tiling, 3 auto without halo staging
    const bool mfma_ok = dtype == MDCNN_F16 && conv_path != 1 && e.Cin % 16 == 0 && e.Cout % 32 == 0;
    if (mfma_ok && conv_path == 0) {
        bool done = false;
        hipError_t err = launch_halo(eb, nb, nseg, alone, st, pick, &done, read);
        if (!done) err = launch_up(eb, nb, st, pick, &done, read);
        if (done) { *cls = kClsConvMfma; return err; }
    }
    // (the tiled kernel addresses deltas and weights with 32-bit byte offsets)
    const bool small32 = (long long)e.sH * e.sW * e.Cin < (1ll << 30) && (long long)e.k * e.k * e.Cin * e.Cout < (1ll << 30);
    if (mfma_ok && (conv_path == 0 || conv_path == 3) && e.Cin % 32 == 0 && small32) {
        *cls = kClsConvMfma;
        if (e.Cin % 128 == 0 && g_kc != 64) return launch_tiled_kc<128>(eb, nb, max_entries, st, pick, read);
        return e.Cin % 64 == 0 ? launch_tiled_kc<64>(eb, nb, max_entries, st, pick, read) : launch_tiled_kc<32>(eb, nb, max_entries, st, pick, read);
    }
    if (pick) return hipSuccess;
    if (mfma_ok) {
        *cls = kClsConvMfma;
        if (e.Cout % 64 == 0)
            k_conv_mfma_f16<2><<<dim3(cap_blocks(nseg * (kSegPixels / 64), 4096), e.Cout / 64, nb), dim3(256), 0, st>>>(eb);
        else
            k_conv_mfma_f16<1><<<dim3(cap_blocks(nseg * (kSegPixels / 128), 4096), e.Cout / 32, nb), dim3(256), 0, st>>>(eb);
        return hipGetLastError();
    }
    if (dtype == MDCNN_F32 && (conv_path == 0 || conv_path == 3) && g_f32_mfma) {
        // 1x1 layers of up to 64 channels and 3x3 layers of 16, whose weights k_conv_mfma_f32 keeps in LDS (1x1, 32 to 64
        // channels at 128 x 128: 7.5 us, 9.0 with k_conv_f32); k_conv_f32 for the rest, 3x3 layers of 32 and 64 channels among
        // them (64 at 128 x 128: 20 us, 35 with the weights in LDS; 32 at 64 x 64: 11.8 and 13.3.  On large windows 32 channels
        // are ahead with the weights in LDS while most pixels are updated - frames in a row of a one-layer network, 512 x 512:
        // 107 us, 146 with k_conv_f32; 128 x 128: 21 and 24 - and behind where updates come in clusters, which this kernel
        // passes over by tiles: a fifth of the frame 90 and 68 us, 256 x 256 38 and 29; five-layer network, 512 x 512 frames,
        // 105 and 99)
        bool done = false;
        const hipError_t err = launch_mfma_f32(eb, nb, nseg, st, &done, read);
        if (done) { *cls = kClsConvMfma; return err; }
        if (f32_applies(e)) { *cls = kClsConvMfma; return launch_conv_f32(eb, nb, st, read); }
    }
    if ((conv_path == 0 || conv_path == 3) && g_f32_mfma && e.k == 3 && e.Cin == 3 && e.Cout % 32 == 0 && e.Cout <= 1024 && !e.up &&
        (long long)e.sH * e.sW * 3 < (1ll << 29)) {
        *cls = kClsConvMfma;
        const unsigned npub = publish_blocks(e, 512), g = cap_blocks(nseg * (kSegPixels / 128), 2048) + npub;
        if (dtype == MDCNN_F16) k_conv_stem_mfma<f16><<<dim3(g, e.Cout / 32, nb), dim3(256), 0, st>>>(npub, g, eb);
        else k_conv_stem_mfma<float><<<dim3(g, e.Cout / 32, nb), dim3(256), 0, st>>>(npub, g, eb);
        return hipGetLastError();
    }
    *cls = kClsConvPlain;
    if ((conv_path == 0 || conv_path == 3) && e.k == 3 && e.Cin == 3 && e.Cout % 32 == 0 && e.Cout <= 256) {
        const int groups = e.Cout / 32, ppb = 256 / groups;
        const size_t smem = (size_t)27 * e.Cout * 4;
        const long long tps = (kSegPixels + ppb - 1) / ppb;
        const unsigned g = cap_blocks(nseg * tps, 2048);
        if (dtype == MDCNN_F16) k_conv_small<f16, 3, 3, 32><<<dim3(g, 1, nb), dim3(256), smem, st>>>(eb, groups, ppb);
        else k_conv_small<float, 3, 3, 32><<<dim3(g, 1, nb), dim3(256), smem, st>>>(eb, groups, ppb);
        return hipGetLastError();
    }
    const int groups = e.Cout / 8;
    if ((conv_path == 0 || conv_path == 3) && e.Cout % 8 == 0 && groups <= 64 && (size_t)e.k * e.k * e.Cin * e.Cout * 4 <= 150 * 1024)
        return dtype == MDCNN_F16 ? launch_ldsw<f16>(eb, nb, max_entries, st) : launch_ldsw<float>(eb, nb, max_entries, st);
    unsigned g = cap_blocks(nseg * (kSegPixels / 16), 8192);
    if (dtype == MDCNN_F16) k_conv_plain<f16><<<dim3(g, 1, nb), dim3(256), 0, st>>>(eb);
    else k_conv_plain<float><<<dim3(g, 1, nb), dim3(256), 0, st>>>(eb);
    return hipGetLastError();
}

}  // namespace mdcnn
