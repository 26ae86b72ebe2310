// Focused convolution on the gfx950 matrix cores (Sec. III-A: a GEMM over the
// kept patches only, with the dense layer's weights).
//
// GEMM view: rows = kept output positions (from the index list), reduction
// K = (tap, input channel), columns = output channels.  The patch matrix is never
// stored: for every (tap, 128-byte chunk of channels) = one pipeline stage, the workgroup
// gathers, for each of its TM positions, the 128 contiguous bytes of that tap's NHWC
// pixel into LDS (zeros where the tap falls outside the image or on an irrelevant
// input pixel), next to the TN x 128-byte slab of weights for the same tap, and feeds
// both to the matrix cores with fp32 accumulators: v_mfma_f32_32x32x16 for bf16 / f16
// storage (64 channels per stage, four instructions per 32 x 32 block), and
// v_mfma_f32_32x32x64_f8f6f4 for 8-bit E4M3 storage (128 channels per stage, two
// instructions of twice the length).  Everything outside the multiply itself - gather,
// swizzle, pipeline, epilogue - moves bytes and is the same code for both.
//
// Data path.  The gathers go straight from global memory into LDS ("buffer_load ...
// lds", 16 bytes per lane) without passing through registers: measured on this chip a
// 128-bit LDS write from registers costs three times a 128-bit LDS read, and staging
// through registers also serialises the workgroup behind bursts of loads.  A wave-wide
// load writes 64 x 16 contiguous bytes of LDS, i.e. 8 tile rows of 128 bytes with no
// padding; bank conflicts on the fragment reads are avoided instead by an XOR swizzle
// applied on the global side: LDS slot c of row r holds the row's 16-byte piece
// c ^ ((r >> 1) & 7).  The loads are issued from inline assembly and waited for with
// explicit s_waitcnt vmcnt(N), so that NB-1 stages stay in flight while one is being
// multiplied (left to itself the compiler drains every outstanding LDS-bound load
// before each LDS read).  A gated lane (padding, irrelevant input pixel, channel
// tail, stage past the end) gets an offset that is out of range for its buffer
// descriptor, for which the hardware writes zeros without touching memory; nothing
// in the gather branches.
//
// The weights are the MFMA's A operand (rows = output channel) and the gathered
// activations its B operand (columns = position), so a lane's accumulators hold 4
// consecutive output channels of one position.  The accumulators start from the bias;
// the epilogue rounds once to the output type, applies ReLU, transposes the tile
// through LDS and stores each kept row as whole 16-byte pieces.  The same kernel clears
// the irrelevant rows (the workgroups that have no tile do it).
//
// The launch grid never depends on the kept count: workgroups stride over the tiles
// and read the count on the device.  Layers with few tiles split every tile's reduction
// over several workgroups, which meet through fp32 partial tiles in the workspace; the
// one that arrives last adds them in a fixed order and writes the tile.
#include "fc_dma_util.hpp"
#include <type_traits>
#include <atomic>

namespace fc {

[[maybe_unused]] constexpr int kMaxTaps = 32;                   // tap-valid bits per row live in one 32-bit word

// Bytes of the LDS stage region: NB buffers of (TM + TN) rows for the tap-by-tap loop; with the
// shared-halo loop (SL > 0) also room for two buffers of SL pixel slots and NBW weight buffers.
template <int TM, int TN, int NB, int SL, int NBW>
constexpr size_t dma_stage_region_bytes()
{
    const size_t classic = (size_t)NB * (TM + TN) * 128;
    const size_t halo = SL > 0 ? (size_t)2 * SL * 128 + (size_t)NBW * TN * 128 : 0;
    return classic > halo ? classic : halo;
}

template <int TM, int TN, int NB, int SL, int NBW>
constexpr size_t dma_lds_bytes()
{
    return dma_stage_region_bytes<TM, TN, NB, SL, NBW>() + (size_t)TM * 5 * sizeof(int32_t) +
           (SL > 0 ? (size_t)(TM + 3 * SL + 8) * sizeof(int32_t) : 0);
}

// DT: storage type of x and w; TO: float or a 16-bit carrier; TM x TN: workgroup tile
// (positions x output channels); WM x WN: wave grid inside it; TAPC: 1 (1x1 kernels),
// 9 (3x3 kernels) or 32 (any kernel of up to 32 taps); NB: LDS stage buffers (NB-1
// stages of loads in flight); MINW: waves per SIMD the register budget leaves room for.
//
// SL > 0 (3x3 kernels with unit horizontal stride and dilation only) adds the shared-halo
// loop.  The three horizontal taps of a kept position read the pixels left of, at and right
// of its centre column, and the kept positions of a tile are sorted, so along a run of
// horizontally adjacent kept positions the left pixel of one is the centre pixel of the one
// before it.  The tile therefore lays its pixels out on a line of "slots": one per kept
// position, plus one before the first and one after the last position of every run; position
// r's taps kw = 0, 1, 2 are then slots cs(r) - 1, cs(r), cs(r) + 1.  For every (kernel row,
// 64-channel chunk) the line is gathered into LDS once and multiplied three times, each time
// against the weights of another horizontal tap, which cuts the gathered bytes by up to three.
// A tile whose line would need more than SL slots (a fragmented mask) runs the tap-by-tap
// loop instead.  NBW: LDS buffers for the per-tap weight slabs of the shared-halo loop.
//
// OWN: the 64 x 64 instance for layers with a mask and no list that label their rows themselves (tiles_label_rows).
// The rows of a tile are consecutive positions, the irrelevant ones are stored as zeros, and no reduction is split.
//
// PACK: the reduction is one run of 16-byte pieces, eight a stage (taps_packed): a row of weights is contiguous over taps and channels,
// and a lane, which fetches the same column of every row of a stage, keeps the tap and the place in it of its own piece.  No stage is
// filled up with channels that are not there: 72 -> 200 on 3 x 75 x 101, stride 2, f16, 11 stages instead of 18, 12.8 -> 10.1 us.
//
// LIST (conv_list_tiles): the list is given and its length, list_rows, known already.
//
// CMP: the instances that serve compacted activations (FC_COMPACT_IN / FC_COMPACT_OUT: rows
// stored in list order).  Separate instances, so that the ordinary ones do not change by a
// register: the 128 x 64 three-buffer instance loses 20 % with a handful more.
template <int DT, typename TO, int TM, int TN, int WM, int WN, int TAPC, int NB, int MINW, int SL, int NBW, bool CMP, bool OWN, bool PACK>
__global__ __launch_bounds__(WM *WN * 64, MINW) void k_conv_dma(Geom g, const uint16_t *__restrict__ x, const uint8_t *__restrict__ mask_in,
                                                                 const uint8_t *__restrict__ mask_out, const uint16_t *__restrict__ w,
                                                                 const float *__restrict__ bias, const int32_t *__restrict__ idx,
                                                                 const int32_t *__restrict__ count, TO *__restrict__ out,
                                                                 float *__restrict__ partials, int32_t *__restrict__ tile_counters)
{
    constexpr bool LIST = false;
    constexpr int list_rows = 0;
#include "fc_conv_dma_body.hpp"
}

// The tap-by-tap loop over the tiles of a list of list_rows rows.
template <int DT, typename TO, int TM, int TN, int WM, int WN, int TAPC, int NB, bool CMP>
__device__ __forceinline__ void conv_list_tiles(const Geom &g, const uint16_t *__restrict__ x, const uint8_t *__restrict__ mask_in,
                                                const uint8_t *__restrict__ mask_out, const uint16_t *__restrict__ w,
                                                const float *__restrict__ bias, const int32_t *__restrict__ idx,
                                                const int32_t *__restrict__ count, int list_rows, TO *__restrict__ out)
{
    constexpr int SL = 0, NBW = 2;
    constexpr bool OWN = false, LIST = true, PACK = false;
    float *const partials = nullptr;
    int32_t *const tile_counters = nullptr;
#include "fc_conv_dma_body.hpp"
}

// Long reductions, tap by tap, of about a tile per CU: one workgroup per CU with two or three stages on their way (two workgroups with one
// stage each wait a round trip a stage), its tile chosen by the kept count, which is known here only, so that one round of tiles
// covers the rows (cus: workgroups that run at once): 128 x 128, in 1x1 layers 192 x 128 where that is more than one round, in 3x3
// layers 128 x 64 where that is still one.  bf16, chained, us at a kept share of 0.1 / 0.3 / 0.5 / 0.7 / 0.9 / 1, two workgroups per CU -> here:
// 1x1 2048 -> 512 on 32 x 15 x 20 18.5 / 25.0 / 27.8 / 32.1 / 35.2 / 35.3 -> 19.5 / 20.6 / 21.2 / 22.3 / 27.4 / 27.9, 1024 -> 512 11.2 / 14.0 / 16.2 / 18.5 /
// 20.0 / 20.0 -> 12.0 / 12.8 / 13.6 / 14.5 / 17.2 / 17.6; 3x3, stride 2, 512 -> 512 from 32 x 29 x 39 33.2 / 34.1 / 62.7 / 69.6 / 104 / 105 -> 30.7 / 33.0 / 41.3 /
// 42.4 / 83 / 84, 256 -> 256 from 9 x 73 x 119 19.1 / 20.5 / 33.0 / 39.3 / 58.5 / 58.0 -> 17.6 / 19.7 / 24.3 / 25.2 / 47.8 / 48.3.  With 128 x 128 tiles
// alone the ends of the range lost: 25.4 at 0.9 kept (1024 -> 512), 38.2 and 22.3 at 0.1 (3x3).
constexpr int kDeepBuffersNarrow = 4, kDeepBuffers = 4, kDeepBuffersTall = 3;
template <int TAPC> constexpr size_t deep_lds_bytes()
{
    constexpr size_t a = dma_lds_bytes<128, 128, kDeepBuffers, 0, 2>();
    constexpr size_t b = TAPC == 1 ? dma_lds_bytes<192, 128, kDeepBuffersTall, 0, 2>() : dma_lds_bytes<128, 64, kDeepBuffersNarrow, 0, 2>();
    return a > b ? a : b;
}

template <int DT, typename TO, int TAPC, bool CMP>
__global__ __launch_bounds__(256, TAPC == 1 ? 1 : 2) void k_conv_deep(Geom g, int cus, const uint16_t *__restrict__ x, const uint8_t *__restrict__ mask_in,
                                                      const uint8_t *__restrict__ mask_out, const uint16_t *__restrict__ w,
                                                      const float *__restrict__ bias, const int32_t *__restrict__ idx,
                                                      const int32_t *__restrict__ count, TO *__restrict__ out)
{
    const int rows = __builtin_amdgcn_readfirstlane(*count), rows128 = (rows + 127) / 128;
    if constexpr (TAPC == 1) {
        if (rows128 * ((g.c_out + 127) / 128) > cus) {
            conv_list_tiles<DT, TO, 192, 128, 2, 2, TAPC, kDeepBuffersTall, CMP>(g, x, mask_in, mask_out, w, bias, idx, count, rows, out);
            return;
        }
    } else {
        if (rows128 * ((g.c_out + 63) / 64) <= cus) {
            conv_list_tiles<DT, TO, 128, 64, 2, 2, TAPC, kDeepBuffersNarrow, CMP>(g, x, mask_in, mask_out, w, bias, idx, count, rows, out);
            return;
        }
    }
    conv_list_tiles<DT, TO, 128, 128, 2, 2, TAPC, kDeepBuffers, CMP>(g, x, mask_in, mask_out, w, bias, idx, count, rows, out);
}

// ---------------------------------------------------------------------------

// The instances a layer can take, by the tile of a workgroup (rows x channels).
struct TileShape {
    enum Kind {
        own64,      // 64 x 64, rows labelled by the tile itself (tiles_label_rows)
        small64,    // 64 x 64, four stage buffers
        line128,    // 128 x 128 on the shared pixel line
        line64,     // 128 x 64 on the shared pixel line
        deep,       // k_conv_deep: one workgroup per CU, the tile by the kept count
        wide128,    // 128 x 128, two workgroups per CU
        narrow64,   // 128 x 64, three workgroups per CU
        tall64,     // 128 x 64, two workgroups per CU
    } kind;
    bool packed; // taps_packed, for tiles that go tap by tap
    int rows() const { return kind == own64 || kind == small64 ? 64 : 128; }
    int cols() const { return kind == line128 || kind == deep || kind == wide128 ? 128 : 64; }
};

// splits: the call brings split-K scratch; labels_rows: a mask and no list
static inline TileShape::Kind choose_kind(const Geom &g, int in_dtype, bool masked, bool labels_rows, bool splits, bool packed)
{
    const bool k1 = g.kh == 1 && g.kw == 1, k3 = g.kh == 3 && g.kw == 3;
    const int64_t rows128 = (g.m + 127) / 128;
    const int64_t tiles128 = rows128 * ((g.c_out + 127) / 128), tiles64 = rows128 * ((g.c_out + 63) / 64);
    if (labels_rows && tiles_label_rows(g, in_dtype)) return TileShape::own64;
    // Layers with only a handful of tiles (the late layers of a network at batch 1) are all
    // latency: 64 x 64 tiles put them on more CUs and four stage buffers keep three gathers in
    // flight (a ResNet-18 stack at batch 1: 0.243 -> 0.221 ms dense, 0.266 -> 0.245 ms focused)
    if (tiles64 <= kSmallLayerTiles) return TileShape::small64;
    // 128 x 128 tiles when there are enough of them to give every CU two workgroups;
    // otherwise 128 x 64, which doubles the tile count (the kept count is not known here,
    // so the dense row count decides)
    //
    // 3x3 kernels that step one pixel at a time horizontally share the gathered pixels
    // between their three horizontal taps (worth it when image rows are long enough for runs
    // of adjacent kept positions; narrow layers with many tiles do better with three
    // workgroups per CU, see below)
    if (k3 && g.sw == 1 && g.dw == 1 && g.wo >= 16 && !packed) {
        // (with many 128 x 128 tiles it pays down to 16-pixel rows: C512@16 at batch 128 is
        // 13 % faster dense and 17 % faster focused than tap by tap)
        if (g.c_out > 64 && tiles128 >= 512) return TileShape::line128;
        // narrow layers: only with very many tiles (C64@128: -7 % focused, -4..8 % dense from batch
        // 128 on, 16 384 row tiles; at 4 800 row tiles, 64 -> 64 on 32 x 120 x 160 positions, three
        // workgroups per CU, below, are 7 % faster, and at batch 16 as fast)
        const bool many_narrow_tiles = rows128 >= 8192;
        if (g.wo >= 32 && (g.c_out > 64 || splits || many_narrow_tiles)) return TileShape::line64;
        // shorter image rows, wide layers, a few hundred tiles (C512 on 32 x 15 x 20 positions:
        // 66 us dense / 45 us chained against 102 / 49 us tap by tap; with 128 tiles, C512@16 at
        // batch 16, tap by tap stays ahead)
        if (g.c_out > 64 && tiles128 >= 256) return TileShape::line64;
    }
    // (1x1 layers keep the wide tiles down to 256 of them: 2048 -> 512 on 32 x 15 x 20 positions,
    // 300 tiles, 37 us dense / 29 us chained against 51 / 32 us with 128 x 64 tiles)
    // Long reductions, tap by tap: from a 128 x 128 tile per CU on (fewer leave CUs without one) to as many rows as a 192 x 128 tile per CU
    // covers, so that 1x1 layers are one round whatever the mask keeps (1024 -> 512 on 32 x 15 x 25, 376 tiles, 0.1 / 0.5 / 0.9 / 1 kept: 11.2 /
    // 17.5 / 19.4 / 19.5 -> 12.0 / 14.2 / 19.2 / 20.3).  Below twelve stages there is little to keep on its way (at twelve, 768 -> 128 on 28 x 30 x 41,
    // 0.3 / 0.5 / 0.7 / 0.9: 9.6 / 11.7 / 14.9 / 16.7 -> 10.4 / 11.3 / 12.1 / 13.5).
    const int cus = conv_grid_cus(), stages = reduction_stages(g, in_dtype, false);
    if ((k1 || k3) && g.c_out > 64 && masked && !labels_rows && !splits && stages >= 12 && tiles128 >= cus &&
        (int64_t)((g.m + 191) / 192) * ((g.c_out + 127) / 128) <= cus)
        return TileShape::deep;
    if (g.c_out > 64 && tiles128 >= (k1 ? 256 : 512)) return TileShape::wide128;
    // narrow layers with many tiles: two stage buffers, so that three workgroups fit a CU
    // and overlap each other's set-up and epilogue
    if (g.c_out <= 64 && !splits) return TileShape::narrow64;
    return TileShape::tall64;
}

static inline TileShape choose_tile(const Geom &g, int in_dtype, bool masked, bool labels_rows, bool splits)
{
    const bool packed = taps_packed(g, in_dtype, masked);
    const TileShape::Kind kind = choose_kind(g, in_dtype, masked, labels_rows, splits, packed);
    return {kind, packed && kind != TileShape::deep};
}

#if !defined(FC_MFMA_PART) || FC_MFMA_PART == 0
// Does a 3x3 layer with a mask and no list label its rows tile by tile (64 x 64 tiles of consecutive positions,
// irrelevant ones stored as zeros) instead of compacting them in a launch of its own?  While all tiles of the
// layer run at once, dropping the irrelevant rows shortens nothing and the compaction is 4.5 us.  Calls one after
// another, the output tensor included, compacted -> here: 72 -> 200 on 3 x 75 x 101, stride 2 (348 tiles of 18 stages)
// 18.8 -> 16.4 us, 64 -> 64 on 8 x 56 x 56 (392 of 9) 14.5 -> 10.5 us, 128 -> 128 on 8 x 28 x 28 (196 of 18) 16.6 -> 13.7 us,
// whatever the kept share.  From two rounds of tiles on, or with long reductions, the rows left out are worth
// it: 64 -> 128 on 8 x 56 x 56 (784 tiles) 14.4 -> 20 us; 392 tiles of 36 stages gain 1.5 us at a kept share of one half
// and lose as much at one fifth.
// (Such a call never splits a tile's reduction; with the list and a workspace the same layer does where few rows are
// kept, so its last bits can be others there.)
bool tiles_label_rows(const Geom &g, int in_dtype)
{
    const bool packed = taps_packed(g, in_dtype, true), k3 = g.kh == 3 && g.kw == 3;
    if (g.kh * g.kw == 1 || (g.flags & FC_RESIDENT_WEIGHTS) || (!packed && (!k3 || g.m <= kInlineRankPositions))) return false;
    const int stages = reduction_stages(g, in_dtype, packed);
    // (with a list these take the shared-halo loop, whose order of stages is another one)
    if (!packed && g.sw == 1 && g.dw == 1 && g.wo >= 32 && stages > 9) return false;
    const int64_t tiles = (int64_t)((g.m + 63) / 64) * ((g.c_out + 63) / 64);
    return tiles <= kSplitGrid && tiles * stages <= 20 * kSplitGrid;
}

bool dense_layer_splits(const Geom &g, int in_dtype)
{
    // (asked for calls with split-K scratch only)
    const TileShape t = choose_tile(g, in_dtype, false, false, true);
    const int64_t tiles = (int64_t)((g.m + t.rows() - 1) / t.rows()) * ((g.c_out + t.cols() - 1) / t.cols());
    const int stages = reduction_stages(g, in_dtype, t.packed);
    return split_k_splits((int)tiles, kSplitGrid, stages, stages) > 1;
}

bool conv_mfma_supported(const Geom &g, int in_dtype, int out_dtype)
{
    if (in_dtype != FC_BF16 && in_dtype != FC_F16 && in_dtype != FC_FP8) return false;
    // fp8 layers round to bfloat16 (or stay fp32), the 16-bit types keep their own format; all can
    // round to fp8
    if (out_dtype != (in_dtype == FC_FP8 ? FC_BF16 : in_dtype) && out_dtype != FC_F32 && out_dtype != FC_FP8)
        return false;
    const uint64_t es = in_dtype == FC_FP8 ? 1u : 2u;
    if ((g.c_in * es) % 16 != 0 || g.c_out % 8 != 0) return false; // 16-byte gathers, 4-channel stores
    if (out_dtype == FC_FP8 && g.c_out % 16 != 0) return false;     // rows are stored in 16-byte pieces
    if (g.kh * g.kw > kMaxTaps) return false;
    // row origins are packed into signed 16-bit halves
    if (g.h > 16384 || g.w > 16384 || g.ph > 8192 || g.pw > 8192) return false;
    // x and w are each addressed through one buffer descriptor with 32-bit byte offsets
    // (the shared pixel line reads x through a descriptor that starts pad_h rows + pad_w pixels early)
    if (((uint64_t)g.n * g.h * g.w + (uint64_t)g.ph * g.w + g.pw) * g.c_in * es >= kBufferLimit) return false;
    if ((uint64_t)g.c_out * g.kh * g.kw * g.c_in * es >= kBufferLimit) return false;
    return true;
}
#endif

// more than 64 KB of dynamic LDS has to be allowed once per function and device; two
// threads that both find the bit clear both set the attribute, which is harmless
[[maybe_unused]] static hipError_t allow_lds(const void *kern, size_t lds, std::atomic<uint64_t> &devices)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t dev_bit = 1ull << (dev & 63);
    if (!(devices.load(std::memory_order_acquire) & dev_bit)) {
        e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        devices.fetch_or(dev_bit, std::memory_order_release);
    }
    return hipSuccess;
}

template <int DT, typename TO, bool CMP, int TM, int TN, int WM, int WN, int TAPC, int NB, int MINW, int SL = 0, int NBW = 2, bool OWN = false, bool PACK = false>
static hipError_t launch_dma(const Geom &g, const void *x, const uint8_t *mask_in, const uint8_t *mask_out,
                             const void *w, const float *bias, const int32_t *idx, const int32_t *count,
                             void *out, float *partials, int32_t *tile_counters, hipStream_t s)
{
    auto kern = k_conv_dma<DT, TO, TM, TN, WM, WN, TAPC, NB, MINW, SL, NBW, CMP, OWN, PACK>;
    constexpr size_t lds = dma_lds_bytes<TM, TN, NB, SL, NBW>();
    static std::atomic<uint64_t> attr_devices{0};
    const hipError_t e = allow_lds(reinterpret_cast<const void *>(kern), lds, attr_devices);
    if (e != hipSuccess) return e;
    const int64_t max_tiles = (int64_t)((g.m + TM - 1) / TM) * ((g.c_out + TN - 1) / TN);
    const int64_t cap = 256 * 8;
    int blocks = (int)((max_tiles < cap ? max_tiles : cap) + 7) & ~7; // a multiple of the XCD count
    Geom gl = g;
    if (partials && !OWN) {
        blocks = kSplitGrid; // few tiles: enough workgroups for the K-split to fill the chip
        if (splits_of_its_own(g, DT, TM)) gl.flags |= kOneUnitPerCu;
    }
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(WM * WN * 64), lds, s, gl, (const uint16_t *)x, mask_in, mask_out,
                       (const uint16_t *)w, bias, idx, count, (TO *)out, partials, tile_counters);
    return hipGetLastError();
}

template <int DT, typename TO, int TAPC, bool CMP>
static hipError_t launch_deep(const Geom &g, const void *x, const uint8_t *mask_in, const uint8_t *mask_out, const void *w,
                              const float *bias, const int32_t *idx, const int32_t *count, void *out, float *, int32_t *, hipStream_t s)
{
    auto kern = k_conv_deep<DT, TO, TAPC, CMP>;
    constexpr size_t lds = deep_lds_bytes<TAPC>();
    static_assert(lds <= 160 * 1024, "LDS of a CU");
    static std::atomic<uint64_t> attr_devices{0};
    const hipError_t e = allow_lds(reinterpret_cast<const void *>(kern), lds, attr_devices);
    if (e != hipSuccess) return e;
    // 1x1: one round, a workgroup per CU; 3x3: as many as 128 x 128 tiles, those of a second round clear their rows beside the first (512 -> 512
    // from 32 x 29 x 39, 0.9 kept, zero-filled 85.7 -> 82.3 us)
    const int tiles = (int)((g.m + 127) / 128) * ((g.c_out + 127) / 128);
    hipLaunchKernelGGL(kern, dim3(TAPC == 1 ? conv_grid_cus() : (tiles + 7) & ~7), dim3(256), lds, s, g, conv_grid_cus(), (const uint16_t *)x, mask_in, mask_out,
                       (const uint16_t *)w, bias, idx, count, (TO *)out);
    return hipGetLastError();
}

#define FC_ARGS g, x, mask_in, mask_out, w, bias, idx, count, out, partials, tile_counters, s

template <int DT, typename TO, int TAPC, bool CMP, bool PACK>
static hipError_t launch_tile(const Geom &g, const void *x, const uint8_t *mask_in, const uint8_t *mask_out,
                              const void *w, const float *bias, const int32_t *idx, const int32_t *count,
                              void *out, float *partials, int32_t *tile_counters, hipStream_t s, TileShape::Kind kind)
{
    switch (kind) {
    case TileShape::own64:
        // (kernels other than 3x3 label their own rows only with packed taps)
        if constexpr ((TAPC == 9 || (TAPC == 32 && PACK)) && !CMP) return launch_dma<DT, TO, CMP, 64, 64, 2, 2, TAPC, 4, 2, 0, 2, true, PACK>(FC_ARGS);
        break;
    case TileShape::small64:
        return launch_dma<DT, TO, CMP, 64, 64, 2, 2, TAPC, 4, 2, 0, 2, false, PACK>(FC_ARGS);
    case TileShape::line128:
        if constexpr (TAPC == 9 && !PACK) return launch_dma<DT, TO, CMP, 128, 128, 2, 2, TAPC, 2, 2, 160, 2>(FC_ARGS);
        break;
    case TileShape::line64:
        if constexpr (TAPC == 9 && !PACK) return launch_dma<DT, TO, CMP, 128, 64, 2, 2, TAPC, 3, 2, 160, 3>(FC_ARGS);
        break;
    case TileShape::deep:
        if constexpr (TAPC != 32 && !PACK) return launch_deep<DT, TO, TAPC, CMP>(FC_ARGS);
        break;
    case TileShape::wide128:
        return launch_dma<DT, TO, CMP, 128, 128, 2, 2, TAPC, (sizeof(TO) == 4 ? 3 : 2), 2, 0, 2, false, PACK>(FC_ARGS);
    case TileShape::narrow64:
        return launch_dma<DT, TO, CMP, 128, 64, 2, 2, TAPC, 2, 3, 0, 2, false, PACK>(FC_ARGS);
    case TileShape::tall64:
        return launch_dma<DT, TO, CMP, 128, 64, 2, 2, TAPC, 3, 2, 0, 2, false, PACK>(FC_ARGS);
    }
    return hipErrorInvalidValue; // (a tile this kernel size has no instance of: choose_tile names none)
}
#undef FC_ARGS

#define FC_ARGS2 g, x, mask_in, mask_out, w, bias, idx, count, out, partials, tile_counters, s

template <int DT, typename TO, bool CMP>
static hipError_t launch_cmp(const Geom &g, const void *x, const uint8_t *mask_in, const uint8_t *mask_out,
                            const void *w, const float *bias, const int32_t *idx, const int32_t *count,
                            void *out, float *partials, int32_t *tile_counters, hipStream_t s)
{
    const TileShape t = choose_tile(g, DT, mask_in != nullptr, mask_in && !idx, partials != nullptr);
    if (g.kh == 1 && g.kw == 1) return launch_tile<DT, TO, 1, CMP, false>(FC_ARGS2, t.kind);
    if (g.kh == 3 && g.kw == 3)
        return t.packed ? launch_tile<DT, TO, 9, CMP, true>(FC_ARGS2, t.kind) : launch_tile<DT, TO, 9, CMP, false>(FC_ARGS2, t.kind);
    return t.packed ? launch_tile<DT, TO, 32, CMP, true>(FC_ARGS2, t.kind) : launch_tile<DT, TO, 32, CMP, false>(FC_ARGS2, t.kind);
}

// The instances of one storage type, with or without compacted activations.
template <int DT, bool CMP>
static hipError_t launch_part(const Geom &g, int out_dtype, const void *x, const uint8_t *mask_in,
                              const uint8_t *mask_out, const void *w, const float *bias, const int32_t *idx,
                              const int32_t *count, void *out, float *partials, int32_t *tile_counters,
                              hipStream_t s)
{
    if (out_dtype == FC_F32) return launch_cmp<DT, float, CMP>(FC_ARGS2);
    if (out_dtype == FC_FP8) return launch_cmp<DT, uint8_t, CMP>(FC_ARGS2);
    return launch_cmp<DT, uint16_t, CMP>(FC_ARGS2);
}

// The kernel instances are spread over six translation units so that a build can compile them
// side by side: a unit compiled with -DFC_MFMA_PART=p (p = 2 * storage type index + compacted)
// holds the instances of part p, part 0 also the two entry points below; without the macro
// this file is one unit that holds everything.
#define FC_PART_PARAMS                                                                                     \
    const Geom &g, int out_dtype, const void *x, const uint8_t *mask_in, const uint8_t *mask_out,         \
        const void *w, const float *bias, const int32_t *idx, const int32_t *count, void *out,             \
        float *partials, int32_t *tile_counters, hipStream_t s
#define FC_PART_ARGS g, out_dtype, x, mask_in, mask_out, w, bias, idx, count, out, partials, tile_counters, s
hipError_t launch_mfma_bf16(FC_PART_PARAMS);
hipError_t launch_mfma_bf16_compact(FC_PART_PARAMS);
hipError_t launch_mfma_f16(FC_PART_PARAMS);
hipError_t launch_mfma_f16_compact(FC_PART_PARAMS);
hipError_t launch_mfma_fp8(FC_PART_PARAMS);
hipError_t launch_mfma_fp8_compact(FC_PART_PARAMS);

#ifndef FC_MFMA_PART
#define FC_MFMA_PART -1
#endif
#define FC_IN_PART(p) (FC_MFMA_PART < 0 || FC_MFMA_PART == (p))

#if FC_IN_PART(0)
hipError_t launch_mfma_bf16(FC_PART_PARAMS) { return launch_part<FC_BF16, false>(FC_PART_ARGS); }
#endif
#if FC_IN_PART(1)
hipError_t launch_mfma_bf16_compact(FC_PART_PARAMS) { return launch_part<FC_BF16, true>(FC_PART_ARGS); }
#endif
#if FC_IN_PART(2)
hipError_t launch_mfma_f16(FC_PART_PARAMS) { return launch_part<FC_F16, false>(FC_PART_ARGS); }
#endif
#if FC_IN_PART(3)
hipError_t launch_mfma_f16_compact(FC_PART_PARAMS) { return launch_part<FC_F16, true>(FC_PART_ARGS); }
#endif
#if FC_IN_PART(4)
hipError_t launch_mfma_fp8(FC_PART_PARAMS) { return launch_part<FC_FP8, false>(FC_PART_ARGS); }
#endif
#if FC_IN_PART(5)
hipError_t launch_mfma_fp8_compact(FC_PART_PARAMS) { return launch_part<FC_FP8, true>(FC_PART_ARGS); }
#endif

#if FC_IN_PART(0)
hipError_t launch_conv_mfma(const Geom &g, int in_dtype, int out_dtype, const void *x, const uint8_t *mask_in,
                            const uint8_t *mask_out, const void *w, const float *bias, const int32_t *idx,
                            const int32_t *count, void *out, float *partials, int32_t *tile_counters,
                            hipStream_t s)
{
    const bool compact = (g.flags & (FC_COMPACT_IN | FC_COMPACT_OUT)) != 0;
    if (in_dtype == FC_BF16) return compact ? launch_mfma_bf16_compact(FC_PART_ARGS) : launch_mfma_bf16(FC_PART_ARGS);
    if (in_dtype == FC_FP8) return compact ? launch_mfma_fp8_compact(FC_PART_ARGS) : launch_mfma_fp8(FC_PART_ARGS);
    return compact ? launch_mfma_f16_compact(FC_PART_ARGS) : launch_mfma_f16(FC_PART_ARGS);
}
#endif

} // namespace fc
