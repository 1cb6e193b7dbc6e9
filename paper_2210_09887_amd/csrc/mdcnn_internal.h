// Internal declarations shared by the host API and the kernel translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include "mdcnn.h"

namespace mdcnn {

// a / d for a >= 0, r = 1 / d within a rounding (rcp_of): below 2^24 the quotient of the floats is off by one at most.  A
// tenth of the instructions of an integer division, of which the start of a tile has one per index it decodes.
__device__ __forceinline__ float rcp_of(int d) { return __builtin_amdgcn_rcpf((float)d); }
__device__ __forceinline__ int fast_div(int a, int d, float r) {
    if (a >= 1 << 24) return a / d;
    const int q = (int)((float)a * r), rem = a - q * d;
    return q + (rem >= d ? 1 : 0) - (rem < 0 ? 1 : 0);
}

// The same for a below 2^24 (a view has at most that many pixels).
__device__ __forceinline__ int div24(int a, int d, float r) {
    const int q = (int)((float)a * r), rem = a - q * d;
    return q + (rem >= d ? 1 : 0) - (rem < 0 ? 1 : 0);
}
// Has these kernel arguments, or what was computed from them alone, in scalar registers at this point.  Left to itself the
// compiler fetches a field of a descriptor where it is used, and every such place is a round trip of its own, one behind the
// other; named together at the start of a kernel they are fetched together.
__device__ __forceinline__ void read_now() {}
template <typename A, typename... R>
__device__ __forceinline__ void read_now(A& a, R&... r);
template <typename A, typename B, typename C, typename D, typename E, typename F, typename G, typename H, typename... R>
__device__ __forceinline__ void read_eight(A& a, B& b, C& c, D& d, E& e, F& f, G& g, H& h, R&... r) {
    asm volatile("" : "+s"(a), "+s"(b), "+s"(c), "+s"(d), "+s"(e), "+s"(f), "+s"(g), "+s"(h));
    read_now(r...);
}
template <typename A, typename... R>
__device__ __forceinline__ void read_now(A& a, R&... r) {
    if constexpr (sizeof...(R) >= 7) {
        read_eight(a, r...);
    } else {
        asm volatile("" : "+s"(a));
        read_now(r...);
    }
}

// A pointer that read_now() has hidden is to global memory all the same: without this its loads are flat ones, which return
// out of order with those of LDS, so that each is waited for by itself.
template <typename T>
__device__ __forceinline__ T* in_global(T* p) {
    auto g = (__attribute__((address_space(1))) T*)p;
    asm("" : "+s"(g));                             // (or the two casts are taken for none)
    return (T*)g;
}

constexpr int kFlagN = 1;   // newly unveiled this frame
constexpr int kFlagU = 2;   // touched by a producer this frame
constexpr int kFlagM = 4;   // updated (emitted a delta) this frame
constexpr int kFlagC = 8;   // was a candidate of step 1 this frame (statistics)
// ring-ordered state of sites with crops, kept across frames
constexpr int kStateUnseen = 1;   // allocated, no frame has covered the pixel yet
constexpr int kStateDirty = 2;    // touched by a producer while outside the crop

// counters[] of a site (int32 slots, device).  Slots [0, 8) are per-frame values of the
// statistics view, filled in where it is read; 64-bit running sums follow (index into
// (unsigned long long*)counters).  All are zeroed when the buffer is first reset.
constexpr int kCntUpdated = 0;      // pixels updated this frame
constexpr int kCntCandidates = 1;   // pixels visited by step 1 this frame
constexpr int kAccUpdated = 4;      // sum of update counts
constexpr int kAccCandidates = 5;   // sum of candidate counts
constexpr int kAccMacs = 6;         // multiply-accumulates of the MFMA kernels into this site (valid taps x Cin x Cout)
constexpr int kAccCompute = 7;      // sum of compute-list lengths of edges into this site
constexpr int kAccMacsPlain = 8;    // multiply-accumulates of the plain-FMA kernels into this site
// The two multiply-accumulate sums are kept as 8 partial sums each (slot + 8 * {1, 2} + block % 8)
// so that the statistics atomics of a launch do not all hit one address.
constexpr int kAccMacsSpread = 16;  // [16, 24): MFMA partials, [24, 32): plain partials
constexpr int kNumCounters = 64;

// Lists are compacted per segment of kSegPixels consecutive linear indices:
// entries of segment g sit at list[g * kSegPixels ...], their number in cnt[g].
// Concatenating the segments in order gives the ascending list.
constexpr int kSegPixels = 256;      // = threads per block: one index per thread

// Device-side view of one site, passed to kernels by value.
struct SiteDev {
    void* A;              // ring H x W x C
    void* P;              // ring Hp x Wp x C
    uint8_t* flags;       // H*W, view order
    void* delta;          // H x W x C, view order
    int* list;            // H*W, segment-local compaction of the update mask
    int* lcnt;            // per segment of list: [2g] entries, [2g+1] candidates of step 1 (this frame)
    unsigned long long* lacc;   // per segment: running sums of the two since the first reset
    int* clist;           // Hp*Wp, segment-local compute list of the last producer
    int* ccnt;            // entries per segment of clist
    unsigned long long* cacc;   // per segment: running sum of compute-list entries
    int* counters;        // kNumCounters
    const float* bias;    // C floats or nullptr
    void* Y;              // ring H x W x C: previous max-pooling output (pool_prev sites), else nullptr
    int H, W, C, Hp, Wp;
    int by0, bx0;         // border before the view (rows, cols)
    int a_oy, a_ox;       // physical ring position of view pixel (0,0) in A
    int p_oy, p_ox;       // physical ring position of window pixel (0,0) in P
    float theta;
    int relu;
    int kind;
    int dtype;
    // Sites with crops (H, W < 65536).  s_off: their state ring S (H x W bytes, kStateUnseen | kStateDirty per
    // pixel, ring order of A) as an offset from A in units of 256 bytes, 0: no crops.  cy, cx: the rows / columns
    // of the view the frame covers, first in the low and end in the high 16 bits (whole view by default).
    unsigned s_off, cy, cx;
    __host__ __device__ uint8_t* S() const { return s_off ? (uint8_t*)A + (size_t)s_off * 256 : nullptr; }
    __host__ __device__ int cy0() const { return (int)(cy & 0xffffu); }
    __host__ __device__ int cy1() const { return (int)(cy >> 16); }
    __host__ __device__ int cx0() const { return (int)(cx & 0xffffu); }
    __host__ __device__ int cx1() const { return (int)(cx >> 16); }
};

// Destination of a residual skip fused into step 1 of its source site: the delta
// a pixel emits is also added to the pending ring of the destination (same view
// shape, same channels) and the pixel is marked touched there.  P == nullptr: none.
struct SkipDev {
    void* P;
    uint8_t* dflags;          // nullptr for OUTPUT sites
    int Hp, Wp, by0, bx0, p_oy, p_ox;
};

// Initialisation job of one site for one camera shift: everything outside the
// kept rectangle of the padded window gets P = bias, everything outside the
// kept rectangle of the view gets A = 0 and flag N.
struct FillJob {
    void* A;
    void* P;
    uint8_t* flags;
    const float* bias;
    int* counters;
    unsigned long long* lacc;   // per-segment running sums, cleared on the first reset
    unsigned long long* cacc;
    int* lcnt;                  // per-segment counts of the frame (n_lacc / n_cacc entries), cleared with them:
    int* ccnt;                  // a site no edge publishes a compute list for must still read as empty
    unsigned s_off, y_off;      // S and Y of the site as offsets from A in units of 256 bytes (0: none): pixels that
                                // enter the view get S = unseen and Y = 0
    int n_lacc, n_cacc;
    int H, W, C, Hp, Wp;
    int a_oy, a_ox, p_oy, p_ox;
    int py0, py1, px0, px1;     // kept rows / cols of the padded window (empty: all new)
    int ay0, ay1, ax0, ax1;     // kept rows / cols of the view
    int nP, nA;                 // pixels to initialise in P / in A
    int dtype;
    int reset_counters;         // 1: first reset of the site, clear its counters and lists
    int per_block;              // items a block initialises
    int flags_only;             // 1: the view's new pixels get their flag N and nothing else - the frame that follows replaces
                                // their accumulated values without reading them
};
// Blocks of a launch that holds several jobs: job j has those from begin[j] on, unused entries are the largest number.  The
// numbers stand side by side because a block's first step is to look for its own: one scalar load and a comparison each,
// where a walk from job to job is a load per job that waits for the last: HRNet-like 384 x 288 frame 611 -> 565 us, 8 videos of
// it 1229 -> 1162.
template <int N>
struct JobBlocks {
    unsigned begin[N];
    unsigned total;
    __host__ void clear() {
        for (unsigned& b : begin) b = ~0u;
        total = 0;
    }
    __host__ void add(int j, unsigned blocks) {
        begin[j] = total;
        total += blocks;
    }
    __device__ __forceinline__ int find(unsigned blk, unsigned* rel) const {
        int j = 0;
        unsigned b0 = begin[0];
#pragma unroll
        for (int k = 1; k < N; ++k) {
            const bool on = blk >= begin[k];
            j = on ? k : j;
            b0 = on ? begin[k] : b0;
        }
        *rel = blk - b0;
        return j;
    }
};
// The same for a launch whose begins come as numbers of their own, the first arguments of the kernel (b0 is 0): those the command
// processor leaves in scalar registers (build flag amdgpu-kernarg-preload-count), and the job's descriptor is the first thing a block asks memory for.
__device__ __forceinline__ int find_job(unsigned b1, unsigned b2, unsigned b3, unsigned b4, unsigned b5, unsigned blk, unsigned* rel) {
    int j = 0;
    unsigned b0 = 0;
    auto next = [&](int k, unsigned b) {
        const bool on = blk >= b;
        j = on ? k : j;
        b0 = on ? b : b0;
    };
    next(1, b1);
    next(2, b2);
    next(3, b3);
    next(4, b4);
    next(5, b5);
    *rel = blk - b0;
    return j;
}
constexpr int kMaxFillJobs = 20;
struct FillBatch {
    JobBlocks<kMaxFillJobs> blocks;
    FillJob j[kMaxFillJobs];
    int n;
};
// 16-byte chunks (or single elements) a block initialises.  A full reset is a plain fill, bound by the
// number of blocks; after a camera shift a block's time is latency (bias loads, ring arithmetic per item), so
// the strips get more, smaller blocks.
constexpr int kFillItemsPerBlockFull = 2048, kFillItemsPerBlockStrip = 512;
inline unsigned fill_blocks(const FillJob& j) {   // blocks a job takes in a launch (none if nothing was unveiled)
    const int vec = j.dtype == MDCNN_F16 ? 8 : 4;
    const int chunks = j.C % vec == 0 ? j.C / vec : j.C;
    const long long items = (long long)j.nP * chunks + (long long)j.nA * (j.flags_only ? 1 : chunks);
    const long long blocks = (items + j.per_block - 1) / j.per_block;
    return (unsigned)(blocks < 1 && j.reset_counters ? 1 : blocks);
}
static_assert(sizeof(FillBatch) <= 4000, "kernel arguments stay below 4 KiB");

// One edge as seen by the list and convolution kernels.
struct EdgeDev {
    // source
    const void* delta;
    const uint8_t* sflags;
    int* pub_list;            // non-null on the one edge of a forward call that also compacts
    int* pub_lcnt;            //   the source's update mask into its list L (segment-local)
    unsigned long long* pub_lacc;
    int* scounters;
    int sH, sW, Cin;
    // destination
    void* P;
    uint8_t* dflags;          // nullptr for OUTPUT sites
    int* clist;
    int* ccnt;
    unsigned long long* cacc;
    int* dcounters;
    int dH, dW, Cout, Hp, Wp, by0, bx0, p_oy, p_ox;
    // operator
    const void* w;            // [tap][cout][cin]
    const void* wp;           // the same weights packed [tap][cin/16][cout][16], or nullptr
    int k, stride, pad, up;
    // max pooling (op == 1; op == 2: the previous output of a reset pixel was zeroed with it): the source's
    // accumulated ring and the destination's previous outputs.
    // Truncation-free destination (op == 3, 1x1 convolution): there is no P; dY is the destination's
    // accumulated ring A (addressed with d_aoy, d_aox), sA its delta map (view order, written here),
    // wp its bias (floats, or nullptr) and s_relu its activation.
    // Convolution (op == 0): dY is where the launch also writes f(P) of the destination's view, s_relu that activation, or
    // nullptr (the last edge into an OUTPUT site, kernels that launch_conv says do it).
    const void* sA;
    void* dY;
    int s_aoy, s_aox, s_relu, d_aoy, d_aox, op;
};
constexpr int kOpTruncFree = 3;
// Blocks of a launch that publish the lists of an edge (publish_edge): a segment of either list per wave, at most `cap` blocks.
inline unsigned publish_blocks(const EdgeDev& e, int cap = 128) {
    const long long nsrc = e.pub_list ? ((long long)e.sH * e.sW + kSegPixels - 1) / kSegPixels : 0;
    const long long ndst = e.up ? 0 : ((long long)e.Hp * e.Wp + kSegPixels - 1) / kSegPixels;
    if (nsrc + ndst == 0) return 0;
    const long long b = ((nsrc > ndst ? nsrc : ndst) + 3) / 4;
    return (unsigned)(b < 1 ? 1 : b > cap ? cap : b);
}

// Blocks of an edge that reads its destination out (read_rest): 2048 pieces of 16 bytes each, at most 256 pixels.
constexpr int kCopyPieces = 2048;
__host__ __device__ inline int copy_pixels(int pieces) { return pieces >= kCopyPieces ? 1 : kCopyPieces / pieces < 256 ? kCopyPieces / pieces : 256; }
inline unsigned copy_blocks(const EdgeDev& e, int esize) {
    if (e.op || !e.dY) return 0;
    const int ppb = copy_pixels(e.Cout * esize / 16);
    return (unsigned)((e.dH * e.dW + ppb - 1) / ppb);
}

// Several independent streams (same network, own buffers and camera paths) share
// one launch: blockIdx.z picks the stream.  The descriptors travel as kernel
// arguments (4 KiB at most), hence the limit.
constexpr int kMaxBatch = 16;
struct EdgeBatch { EdgeDev d[kMaxBatch]; };
struct Step1Batch {
    SiteDev s[kMaxBatch];
    SkipDev skip[kMaxBatch];
    const void* X[kMaxBatch];
    const uint8_t* forced[kMaxBatch];
};
// One site's step 1 and, in the same launch, initialisation jobs of OTHER sites that nothing in this
// launch touches (the first blocks of the grid; the site's own blocks follow).
// own: the site's own initialisation (an INPUT site without crops, not its first reset), done by step 1 itself - a pixel
// outside the kept rectangle of the view counts as newly unveiled and its accumulated value as zero.
constexpr int kMaxRiders = 18;
struct Step1Fill {
    SiteDev s;
    SkipDev skip;
    const void* X;
    const uint8_t* forced;
    FillJob own;
    int has_own;
    int n;
    JobBlocks<kMaxRiders> blocks;
    FillJob j[kMaxRiders];
};
static_assert(sizeof(Step1Fill) <= 4000, "kernel arguments stay below 4 KiB");
static_assert(sizeof(EdgeBatch) <= 3800 && sizeof(Step1Batch) <= 3800, "kernel arguments stay below 4 KiB");

enum KernelClass { kClsShift = 0, kClsStep1, kClsLists, kClsConvMfma, kClsConvPlain, kClsIdentity, kClsReadout, kClsPool, kNumClasses };

hipError_t launch_shift_fill(const FillBatch& fb, hipStream_t st);
// n streams; geometry and dtype are those of stream 0 (the host checks that all agree)
hipError_t launch_step1(const Step1Batch& b, int n, hipStream_t st);
// fills in blocks
hipError_t launch_step1_fill(Step1Fill& a, hipStream_t st);
// Tile configurations k_conv_multi carries: -1, or the number of the body.  They are the small ones - tiles of at most
// half a list segment - plus the 64- and 128-pixel gather tiles: an edge that takes larger tiles fills the GPU by itself.
constexpr int kMultiRectBodies = 15, kMultiHaloBodies = 2, kMultiTiledBodies = 15;
constexpr int kMultiUpBody = kMultiRectBodies + kMultiHaloBodies + kMultiTiledBodies, kMultiListBody = kMultiUpBody + 1;      // (the last: lists only, no tiles)
constexpr int kRectS2One = 1, kRectS2 = 2, kRectS2Half = 3;      // the stride-2 tiles, in place of their entries
constexpr int multi_rect_body(int m, int tn) {
    return m == 64 || m == 96 || m == 128 ? (m / 32 - 2) * 2 + tn - 1 : m >= kRectS2One && m <= kRectS2Half ? 6 + (m - 1) * 3 + tn / 2 : -1;
}
constexpr int multi_halo_body(int nsub, int wmv, int wk, int tm, int tn, int kc, int nld, int ring, bool t2d) {
    const int c[kMultiHaloBodies][9] = {{2, 2, 2, 2, 1, 32, 3, 3, 1}, {4, 2, 2, 1, 1, 32, 2, 9, 1}};
    for (int i = 0; i < kMultiHaloBodies; ++i)
        if (c[i][0] == nsub && c[i][1] == wmv && c[i][2] == wk && c[i][3] == tm && c[i][4] == tn && c[i][5] == kc && c[i][6] == nld &&
            c[i][7] == ring && (c[i][8] != 0) == t2d)
            return kMultiRectBodies + i;
    return -1;
}
constexpr int multi_tiled_body(int wm, int wn, int tm, int tn, int kc, int pipe) {
    const int c[5][4] = {{2, 2, 1, 1}, {4, 1, 1, 1}, {2, 2, 2, 1}, {2, 2, 1, 2}, {2, 2, 2, 2}};
    for (int i = 0; i < 5; ++i)
        if (pipe == 1 && c[i][0] == wm && c[i][1] == wn && c[i][2] == tm && c[i][3] == tn)
            return kMultiRectBodies + kMultiHaloBodies + 3 * i + (kc == 32 ? 0 : kc == 64 ? 1 : 2);
    return -1;
}
// How the tiles of an edge are dealt to its blocks.  per_*: 2^32 / divisor, rounded up, 0 for 1 (by_reciprocal).
struct TileGrid {
    unsigned npub;            // blocks that publish the lists
    unsigned ncopy;           // blocks that read out what the tiles leave alone, the last of the edge (read_rest)
    int NT;                   // cout tiles
    int p0, p1;               // rectangular tiles: rows, columns; gather tiles: xcd_map
    int tiles_x;              // rectangles in a row
    unsigned per_NT, per_tiles_x;
    int early;                // upsampling tiles: everything is requested at once
};
// How launch_conv would run an edge; body < 0: not with one of those configurations.
struct ConvPick {
    int body, items;
    TileGrid g;
    unsigned blocks, smem;    // blocks of the edge
};

// Several edges that do not depend on each other in one launch.  The videos of a batch have their sites at different
// addresses and ring origins and everything else in common, so a job carries the descriptor of the first video and a
// video what differs: the distance of its source and destination memory and the origin of the destination's P.
constexpr int kMaxMultiJobs = 6, kMaxConvVids = 96, kMaxStep1Vids = 48;
struct ConvJob {
    EdgeDev e;
    int body, items;
    TileGrid g;
    unsigned blocks;          // its blocks of the grid (their numbers start at a multiple of 8, for the XCDs)
};
struct ConvVid {
    long long sd, dd;
    int p_oy, p_ox;
};
struct ConvMulti {
    JobBlocks<kMaxMultiJobs> blocks;
    int n, videos;
    ConvJob job[kMaxMultiJobs];
    ConvVid vid[kMaxConvVids];    // job j, video b: vid[j * videos + b]
};
static_assert(sizeof(ConvMulti) <= 4000, "kernel arguments stay below 4 KiB");
hipError_t launch_conv_multi(ConvMulti& m, int videos, unsigned smem, hipStream_t st);      // fills in blocks and videos

// The same for step 1 of several sites (PREACT sites only: an INPUT site takes a frame).  The job holds what networks of
// equal shape have in common and the addresses of the first video, everything else is the video's own.
struct Step1Job {
    void *A, *P, *delta;
    uint8_t* flags;
    void* skip_P;             // destination of the residual add, nullptr: none
    uint8_t* skip_flags;
    int H, W, C, Hp, Wp, by0, bx0, relu;
    int skip_Hp, skip_Wp, skip_by0, skip_bx0;
};
struct Step1Vid {
    long long sd, kd;         // distance of the site's memory, of the memory of the residual add's destination
    int a_oy, a_ox, p_oy, p_ox, k_oy, k_ox;
    unsigned s_off, cy, cx;   // (where the state ring lies depends on what else the site keeps)
    float theta;
};
struct Step1Multi {
    JobBlocks<kMaxMultiJobs> blocks;
    int n, videos;
    Step1Job job[kMaxMultiJobs];
    Step1Vid vid[kMaxStep1Vids];
};
static_assert(sizeof(Step1Multi) <= 4000, "kernel arguments stay below 4 KiB");
bool step1_multi_applies(const SiteDev& s);
hipError_t launch_step1_multi(Step1Multi& m, int videos, hipStream_t st);      // fills in blocks and videos

// e.k < 0: no operator, only the compaction of the source's update mask.
// returns the kernel class that was launched in *cls
// alone: the launches of other frames do not run beside this one (the choice of the tile, not its results)
// read: set to true if the launch also writes f(P) of the destination's view to EdgeDev::dY (asked for by its not being nullptr)
// pick: nothing is launched; *pick says with which configuration of k_conv_multi the edge would run, if with one
hipError_t launch_conv(const EdgeBatch& eb, int n, int dtype, int conv_path, bool alone, hipStream_t st, int* cls, ConvPick* pick = nullptr, bool* read = nullptr);
// fp32 layers on the matrix cores (kernels_f32.hip): shapes it takes, launch
bool f32_applies(const EdgeDev& e);
hipError_t launch_conv_f32(const EdgeBatch& eb, int nb, hipStream_t st, bool* read);
// host-only: row tiles of a tile of conv_f32s.h
int split_choice(int Hp, int Wp, int Cin, int Cout, int nb);
extern int g_tile, g_pipe, g_xcd, g_kc, g_halo, g_halo_sub, g_f32_mfma;   // convolution tuning knobs
// host-only: the rectangle th x tw of at most `sub` pixels whose halo fits `cap` staged pixels, with the fewest tiles over an Hp x Wp window
bool tile_2d(int Hp, int Wp, int k, int sub, int cap, int* th_out, int* tw_out, long long* tiles_out);
// host-only: rows of 16 source pixels a tile of m entries stages (conv_rect.h), its rectangle, and which tile a launch takes
constexpr int rect_rows(int m) { return m <= 96 ? 10 : m == 128 ? 12 : m == 160 ? 14 : 20; }
void rect_tile(int Hp, int Wp, int m, int rows, int stride, int* th_out, int* tw_out, long long* tiles_out);
// alone: see launch_conv; shared: beside other edges in one launch
void rect_choice(int Hp, int Wp, int Cin, int Cout, int videos, bool alone, bool shared, int* tn, int* m);
// host-only: which tile of the gather kernel a launch takes (MDCNN_OPT_CONV_TILE's number)
int gather_choice(long long entries, int k, int Cout, bool shared);
hipError_t launch_pack_weights(const void* src, void* dst, int taps, int Cout, int Cin, hipStream_t st);
// Post-processed update mask of an INPUT site over the rectangle (y0, x0, Hc, Wc) of its view.
struct MaskJob {
    SiteDev s;
    const void* X;            // Hc x Wc x C, storage dtype
    const float* roi;         // Hc x Wc or nullptr
    uint8_t* mask;            // Hc x Wc
    int y0, x0, Hc, Wc;
    float theta, base, gain;
    int q, suppress, d;
};
constexpr int kMaskMaxDilate = 32;
hipError_t launch_input_mask(const MaskJob& j, hipStream_t st);
hipError_t launch_read_view(const SiteDev& s, int what, void* dst, hipStream_t st);
// The OUTPUT site of n videos of one network in one launch (MDCNN_VIEW_OUT or MDCNN_VIEW_CROP_OUT): 8 videos of the HRNet-like
// network 1100 -> 1079 us a frame of each, eight launches of 4.5 us before.
struct ReadBatch {
    SiteDev s[kMaxBatch];
    void* dst[kMaxBatch];
};
static_assert(sizeof(ReadBatch) <= 3800, "kernel arguments stay below 4 KiB");
hipError_t launch_read_outputs(const ReadBatch& b, int n, int what, hipStream_t st);
hipError_t launch_zero_bytes(void* dst, size_t bytes, hipStream_t st);      // bytes a multiple of 16, dst 16-byte aligned
hipError_t launch_bench_copy(const void* src, void* dst, size_t bytes, hipStream_t st);
hipError_t launch_bench_mfma(float* sink, int iters, int blocks, hipStream_t st);
hipError_t launch_write_view(const SiteDev& s, int what, const void* src, hipStream_t st);

}  // namespace mdcnn
