// Internal declarations shared by the library's translation units (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include "focused_conv.h"

namespace fc {

// n / d for n < 2^31 as a multiply and a shift: s = ceil(log2 d), m = ceil(2^(31+s) / d);
// m*d = 2^(31+s) + e with e < d <= 2^s, so the estimate is off by less than 1/d.
struct FastDiv {
    uint32_t m, s;
};

static inline FastDiv make_fastdiv(uint32_t d)
{
    FastDiv f;
    f.s = 0;
    while ((1ull << f.s) < d) ++f.s;
    f.m = (uint32_t)(((1ull << (31 + f.s)) + d - 1) / d);
    return f;
}

__device__ __forceinline__ uint32_t fast_div(uint32_t n, FastDiv f)
{
    return (uint32_t)(((uint64_t)n * f.m) >> (31 + f.s));
}

// Geometry handed to every kernel (plain ints, passed by value).
struct Geom {
    int32_t n, h, w, c_in, c_out, kh, kw;
    int32_t sh, sw, ph, pw, dh, dw;
    int32_t ho, wo;
    int32_t m;        // n*ho*wo
    uint32_t flags;
    FastDiv div_wo, div_ho;
};

// 16-bit storage types are carried as raw bit patterns.
struct bf16_t { uint16_t bits; };
struct f16_t { uint16_t bits; };

__device__ __forceinline__ float to_float(float v) { return v; }
__device__ __forceinline__ float to_float(bf16_t v) { return __uint_as_float((uint32_t)v.bits << 16); }
__device__ __forceinline__ float to_float(f16_t v)
{
    _Float16 h;
    __builtin_memcpy(&h, &v.bits, 2);
    return (float)h;
}

// float -> storage, round to nearest even (NaN stays NaN).
__device__ __forceinline__ uint16_t bf16_bits_rne(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x0040u);
    return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}
__device__ __forceinline__ uint16_t f16_bits_rne(float f)
{
    _Float16 h = (_Float16)f;
    uint16_t b;
    __builtin_memcpy(&b, &h, 2);
    return b;
}
__device__ __forceinline__ void from_float(float f, float *o) { *o = f; }
__device__ __forceinline__ void from_float(float f, bf16_t *o) { o->bits = bf16_bits_rne(f); }
__device__ __forceinline__ void from_float(float f, f16_t *o) { o->bits = f16_bits_rne(f); }

static inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

constexpr int kCompactBlockThreads = 256;
constexpr int kCompactBlockElems = 4096; // positions per workgroup of the list kernels

static inline int64_t compact_blocks(int64_t m) { return (m + kCompactBlockElems - 1) / kCompactBlockElems; }

// How output positions map to input-mask pixels (centre tap of the receptive field).
struct MaskGeom {
    int32_t n, h, w, ho, wo, sh, sw, ch0, cw0;
    int32_t identity; // output position p reads input pixel p (stride 1, same size, centred)
    int32_t packed_in, packed_out; // the mask read / written is one bit per pixel (see mask_at)
    int64_t m;        // n*ho*wo
};

// Values loaded together: without this the compiler moves each load to the branch that uses it, with a wait of its own there.
template <typename T, int N> __device__ __forceinline__ void loaded_together(T (&v)[N])
{
#pragma unroll
    for (int i = 0; i < N; ++i) __asm__ volatile("" : "+v"(v[i]));
}

// A mask is one byte per pixel (nonzero = relevant) or, packed, one bit per pixel: bit p & 31
// of the 32-bit word p >> 5 (little-endian, so the same bits as bit p & 63 of the 64-bit word
// p >> 6, one wave ballot); bits past the last pixel are zero.
// One load of a byte for both, without a branch: a branch per form ends in a wait for its load, so look-ups that a kernel
// makes together came back one after another.
__device__ __forceinline__ bool mask_at(const uint8_t *__restrict__ m, int64_t p, bool packed)
{
    const uint32_t byte = m[packed ? p >> 3 : p];
    return (byte >> (packed ? (uint32_t)p & 7u : 0u)) & (packed ? 1u : 0xffu);
}

__host__ __device__ static inline MaskGeom mask_geom(int n, int h, int w, int kh, int kw, int sh, int sw, int ph, int pw, int dh,
                                 int dw, int ho, int wo)
{
    MaskGeom g;
    g.n = n; g.h = h; g.w = w; g.ho = ho; g.wo = wo; g.sh = sh; g.sw = sw;
    g.ch0 = -ph + dh * ((kh - 1) / 2);
    g.cw0 = -pw + dw * ((kw - 1) / 2);
    g.identity = (sh == 1 && sw == 1 && ho == h && wo == w && g.ch0 == 0 && g.cw0 == 0) ? 1 : 0;
    g.packed_in = g.packed_out = 0;
    g.m = (int64_t)n * ho * wo;
    return g;
}

// bit j = output position p0 + j is kept (positions at or past g.m read as 0)
__device__ __forceinline__ uint32_t kept_flags16(const MaskGeom &g, const uint8_t *__restrict__ mask_in,
                                                 int64_t p0)
{
    uint32_t flags = 0;
    if (p0 >= g.m) return 0;
    if (g.identity && g.packed_in) {
        // p0 is a multiple of 16: the labels are one 16-bit piece of the packed mask
        flags = reinterpret_cast<const uint16_t *>(mask_in)[p0 >> 4];
        if (p0 + 16 > g.m) flags &= (1u << (uint32_t)(g.m - p0)) - 1u;
        return flags;
    }
    if (g.identity && p0 + 16 <= g.m) {
        const uint4 v = *reinterpret_cast<const uint4 *>(mask_in + p0);
        const uint32_t wds[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int b = 0; b < 4; ++b)
                flags |= ((wds[q] >> (8 * b)) & 0xffu) ? (1u << (4 * q + b)) : 0u;
        return flags;
    }
    // (positions fit 31 bits: 32-bit divisions; addresses first, then all sixteen bytes in
    // flight together)
    const uint32_t t = (uint32_t)p0 / (uint32_t)g.wo;
    int ow = (int)((uint32_t)p0 - t * (uint32_t)g.wo);
    int b = (int)(t / (uint32_t)g.ho);
    int oh = (int)(t - (uint32_t)b * (uint32_t)g.ho);
    int row_at = (b * g.h + min(max(oh * g.sh + g.ch0, 0), g.h - 1)) * g.w;
    int at[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        at[j] = p0 + j < g.m ? row_at + min(max(ow * g.sw + g.cw0, 0), g.w - 1) : -1;
        if (++ow == g.wo) {
            ow = 0;
            if (++oh == g.ho) {
                oh = 0;
                ++b;
            }
            row_at = (b * g.h + min(max(oh * g.sh + g.ch0, 0), g.h - 1)) * g.w;
        }
    }
    if (g.packed_in) {
        uint32_t got[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) got[j] = reinterpret_cast<const uint32_t *>(mask_in)[max(at[j], 0) >> 5];
        loaded_together(got);
#pragma unroll
        for (int j = 0; j < 16; ++j) flags |= (at[j] >= 0 ? (got[j] >> (at[j] & 31)) & 1u : 0u) << j;
        return flags;
    }
    uint32_t got[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) got[j] = mask_in[max(at[j], 0)];
    loaded_together(got);
#pragma unroll
    for (int j = 0; j < 16; ++j) flags |= at[j] >= 0 && got[j] ? (1u << j) : 0u;
    return flags;
}

// label of output position p: its mask_out entry, or the input mask under its centre tap
__device__ __forceinline__ bool position_kept(const Geom &g, const uint8_t *__restrict__ mask_in,
                                              const uint8_t *__restrict__ mask_out, int64_t p)
{
    const bool packed = (g.flags & FC_PACKED_MASKS) != 0;
    if (mask_out) return mask_at(mask_out, p, packed);
    const uint32_t t = (uint32_t)p / (uint32_t)g.wo; // (position counts fit 31 bits)
    const int ow = (int)((uint32_t)p - t * (uint32_t)g.wo);
    const int b = (int)(t / (uint32_t)g.ho);
    const int oh = (int)(t - (uint32_t)b * (uint32_t)g.ho);
    int ih = min(max(oh * g.sh - g.ph + g.dh * ((g.kh - 1) / 2), 0), g.h - 1);
    int iw = min(max(ow * g.sw - g.pw + g.dw * ((g.kw - 1) / 2), 0), g.w - 1);
    return mask_at(mask_in, (int64_t)(b * g.h + ih) * g.w + iw, packed);
}

// Between LDS writes of some lanes of a wave and the reads of others (and the other way round): LDS serves a wave's accesses in
// the order they were issued, and this keeps the compiler to the order they are written in.
__device__ __forceinline__ void wave_lds_order() { __asm__ volatile("" ::: "memory"); }

// Zero-fill of the irrelevant output rows (whole 16-byte pieces, `pieces` per row): wave `worker` of
// `workers` looks at 64 positions at a time (one label each), lists the irrelevant ones in LDS in order
// (`dropped`: 64 ints of its own), and then all its lanes store 16-byte pieces of those rows, so the stores
// are dense and none of them waits for a label.  The labels of the next 64 positions are requested before
// the stores of the current ones.
__device__ __forceinline__ void clear_irrelevant(const Geom &g, const uint8_t *__restrict__ mask_in,
                                                 const uint8_t *__restrict__ mask_out, void *__restrict__ out, int pieces,
                                                 int worker, int workers, int32_t *dropped)
{
    const int lane = threadIdx.x & 63;
    const int64_t step = (int64_t)workers * 64;
    typedef uint32_t u32x4_nt __attribute__((ext_vector_type(4)));
    const u32x4_nt zero4 = {0u, 0u, 0u, 0u};
    u32x4_nt *o4 = reinterpret_cast<u32x4_nt *>(out);
    int64_t p0 = (int64_t)worker * 64;
    bool kept = p0 + lane >= g.m || position_kept(g, mask_in, mask_out, p0 + lane);
    for (; p0 < g.m; p0 += step) {
        const uint64_t drop = __ballot(!kept);
        const int nd = __popcll(drop);
        if (!kept) dropped[__popcll(drop & ((1ull << lane) - 1ull))] = (int32_t)(p0 + lane); // in position order
        wave_lds_order();
        const int64_t pn = p0 + step + lane;
        kept = pn >= g.m || position_kept(g, mask_in, mask_out, pn);
        const int total = nd * pieces;
        for (int c = lane; c < total; c += 64) {
            const int rk = c / pieces, pc = c - rk * pieces;
            __builtin_nontemporal_store(zero4, o4 + (int64_t)dropped[rk] * pieces + pc);
        }
        wave_lds_order();
    }
}

// The same for positions begin .. end - 1 without a list: the rows of 64 positions are one piece of memory, and a lane clears
// those of its 16-byte pieces that lie in irrelevant rows (div_pieces: by the pieces of a row).
__device__ __forceinline__ void clear_irrelevant_runs(const Geom &g, const uint8_t *__restrict__ mask_in, const uint8_t *__restrict__ mask_out,
                                                      void *__restrict__ out, int pieces, const FastDiv &div_pieces, int64_t begin, int64_t end,
                                                      int worker, int workers)
{
    const int lane = threadIdx.x & 63;
    const int64_t step = (int64_t)workers * 64;
    typedef uint32_t u32x4_nt __attribute__((ext_vector_type(4)));
    const u32x4_nt zero4 = {0u, 0u, 0u, 0u};
    u32x4_nt *o4 = reinterpret_cast<u32x4_nt *>(out);
    int64_t p0 = begin + (int64_t)worker * 64;
    bool kept = p0 + lane >= end || position_kept(g, mask_in, mask_out, p0 + lane);
    for (; p0 < end; p0 += step) {
        const uint64_t drop = __ballot(!kept);
        const int64_t pn = p0 + step + lane;
        kept = pn >= end || position_kept(g, mask_in, mask_out, pn);
        if (drop == 0) continue;
        u32x4_nt *at = o4 + p0 * pieces;
        for (int c = lane; c < 64 * pieces; c += 64)
            if ((drop >> fast_div((uint32_t)c, div_pieces)) & 1ull) __builtin_nontemporal_store(zero4, at + c);
    }
}

// inclusive prefix sum over the 64 lanes of a wave, on the cross-lane data path of the
// vector ALU (no LDS traffic): shifts by 1, 2, 4, 8 inside each row of 16 lanes, then the last
// lane of row 0 / row 2 is broadcast into row 1 / row 3, then lane 31 into rows 2 and 3.
__device__ __forceinline__ int wave_inclusive_scan(int v)
{
    // row_shr:n = 0x110 + n (a lane with no source inside its row adds 0)
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);
    // row_bcast:15 into rows 1 and 3 (row mask 0b1010), row_bcast:31 into rows 2 and 3 (0b1100)
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
    return v;
}

// Neighbouring units of work on one XCD: workgroup b runs on XCD b mod 8, so with units dealt in the order of the numbers the pixels that
// neighbours share are fetched by every XCD's L2.  Here XCD j takes the j-th contiguous eighth of the units, or of every 2^lg of them.
// (By shifts: two more arguments, for runs of any length, came to 0.4 us of a launch whose arguments no cache holds.)
__device__ __forceinline__ int xcd_eighth(int block, int grid)
{
    const int xcd = block & 7;
    return xcd * (grid >> 3) + min(xcd, grid & 7) + (block >> 3);
}
constexpr int kOneSegment = 30; // (launches have fewer workgroups)
__device__ __forceinline__ int xcd_eighth_of(int block, int grid, int lg)
{
    const int base = block >> lg << lg;
    return base + xcd_eighth(block - base, min(grid - base, 1 << lg));
}

// ---- launchers (each enqueues on `s`, returns a hipError_t) ----------------
hipError_t launch_mask_downsample(const uint8_t *mask_in, int n, int h, int w, int kh, int kw,
                                  int sh, int sw, int ph, int pw, int dh, int dw, int ho, int wo,
                                  uint8_t *mask_out, hipStream_t s);
// Patch labels by a window rule: any pixel of the window relevant, or all of them.
hipError_t launch_mask_window(const uint8_t *mask_in, int n, int h, int w, int kh, int kw, int sh, int sw,
                              int ph, int pw, int dh, int dw, int ho, int wo, bool all, uint8_t *mask_out,
                              hipStream_t s);
// What the compaction can do on the side for the convolution that follows it.
struct CompactExtras {
    int32_t *zero = nullptr; // zero_n ints to clear (the split-K tile counters)
    int32_t zero_n = 0;
};

// Kept positions of the layer whose mask geometry is g: writes mask_out (0/1 bytes;
// may be NULL), the ascending index list and its length.
hipError_t launch_compact(const MaskGeom &g, const uint8_t *mask_in, uint8_t *mask_out, int32_t *idx,
                          int32_t *count, int32_t *block_counts, const CompactExtras &extras, hipStream_t s);
// Mask pyramid: level l is the centre-tap rescaling of level l - 1, level 0 that of the input mask.
constexpr int kMaxPyramidLevels = 8;

// A level's coordinate -> the input mask's, along one axis: clamp(v * mul + add, lo, hi).  Rescaling steps
// are such maps, and so is a composition of them (a clamped value's image is its image, clamped to the
// images of the bounds), so a level reads the input mask with one multiply-add whatever its depth.
struct AxisMap {
    int32_t mul, add, lo, hi;
};
// step v -> clamp(v * stride + first, 0, inner_size - 1), followed by `inner`
AxisMap compose_axis(int32_t stride, int32_t first, int32_t inner_size, const AxisMap &inner);

// One list to build: positions 0 .. m - 1 (flat [n][hl][wl] order), their labels in a mask of h0 x w0 images.
struct LabelMap {
    int32_t m, hl, wl, h0, w0;
    int32_t identity;              // position p reads mask pixel p
    int32_t packed_in, packed_out; // one bit per pixel (see mask_at)
    int32_t block0;                // first workgroup of this list
    AxisMap row, col;
    FastDiv div_w, div_h;
    uint8_t *mask_out;             // the labels, or NULL
    int32_t *idx, *count;
};
template <int NL> struct ListArgs {
    int32_t lists, blocks;
    int32_t vec_in; // the input mask's address allows 16-byte loads
    LabelMap at[NL];
    CompactExtras ex;
};
// block_counts: one int per 4096 positions of every list (not used when the lists are short)
hipError_t launch_lists(const ListArgs<1> &a, const uint8_t *mask_in, int32_t *block_counts, hipStream_t s);
hipError_t launch_lists(const ListArgs<kMaxPyramidLevels> &a, const uint8_t *mask_in, int32_t *block_counts, hipStream_t s);
// kept positions of a [n][ho][wo] mask in tile order; block_counts: one int per 256 tile rows
hipError_t launch_compact_tiled(const uint8_t *mask, int n, int ho, int wo, int tile_h, int tile_w, int32_t *idx,
                                int32_t *count, int32_t *block_counts, hipStream_t s);
constexpr int kMaxListTileWidth = 32; // a tile row's labels are one 32-bit word
static inline int64_t tiled_rows(int n, int ho, int wo, int tile_h, int tile_w)
{
    return (int64_t)n * ((ho + tile_h - 1) / tile_h) * ((wo + tile_w - 1) / tile_w) * tile_h;
}
// bytes -> bits (nonzero byte = 1; the bits of the last word past m are zero), and the
// centre-tap rescaling of a mask in either form into either form
hipError_t launch_mask_pack(const uint8_t *mask, int64_t m, uint64_t *bits, hipStream_t s);
hipError_t launch_mask_rescale(const MaskGeom &g, const uint8_t *mask_in, uint8_t *mask_out, hipStream_t s);
hipError_t launch_zero_fill(const Geom &g, const uint8_t *mask_in, const uint8_t *mask_out, void *out,
                            int out_dtype, hipStream_t s);
hipError_t launch_expand_group_weights(const void *wg, int c_in, int c_out, int taps, int groups, int esize,
                                       void *wd, hipStream_t s);
// keep: [n][ho][wo] bytes or NULL; positions with a zero byte are written as +0 and not computed
hipError_t launch_maxpool(const void *x, int n, int h, int w, int c, int dtype, int k, int stride,
                          int pad, int ho, int wo, const uint8_t *keep, void *out, hipStream_t s);

// Direct convolution over the active rows; any shape, any dtype.  groups > 1: g.c_in / g.c_out
// are the channels of one group, x and out hold all groups side by side.
hipError_t launch_conv_direct(const Geom &g, int in_dtype, int out_dtype, const void *x,
                              const uint8_t *mask_in, const void *w, const float *bias,
                              const int32_t *idx, const int32_t *count, void *out, hipStream_t s, int groups = 1);

// fp32 storage and grouped layers of 16-bit storage on the matrix cores (see fc_conv_reg.hip).  With a
// mask and no list the kernels label positions themselves (from mask_out, or the centre tap of mask_in)
// and clear the irrelevant rows; with a list the caller clears them.
bool conv_f32_supported(const Geom &g);
hipError_t launch_conv_f32(const Geom &g, const void *x, const uint8_t *mask_in, const uint8_t *mask_out, const void *w,
                           const float *bias, const int32_t *idx, const int32_t *count, void *out, hipStream_t s);
bool conv_grouped_supported(const Geom &g, int groups, int in_dtype, int out_dtype);
hipError_t launch_conv_grouped(const Geom &g, int groups, int in_dtype, int out_dtype, const void *x, const uint8_t *mask_in,
                               const uint8_t *mask_out, const void *w, const float *bias, const int32_t *idx,
                               const int32_t *count, void *out, hipStream_t s);

// Depthwise layer (one filter per channel); labels positions from mask_in itself and clears
// the irrelevant rows.
bool conv_depthwise_supported(const Geom &g, int in_dtype);
hipError_t launch_conv_depthwise(const Geom &g, int in_dtype, int out_dtype, const void *x, const uint8_t *mask_in,
                                 const void *w, const float *bias, void *out, hipStream_t s);

// Matrix-core path for layers with at most 4 input channels (RGB stems); clears the irrelevant rows too.
bool conv_stem_supported(const Geom &g, int in_dtype, int out_dtype);
hipError_t launch_conv_stem(const Geom &g, int in_dtype, int out_dtype, const void *x, const uint8_t *mask_in,
                            const uint8_t *mask_out, const void *w, const float *bias, const int32_t *idx,
                            const int32_t *count, void *out, hipStream_t s);

// Split-K scratch of the matrix-core path (optional): fp32 partial tiles and one counter
// per tile.  Only layers with few tiles use it; for the others the sizes are zero.
constexpr int kInlineRankPositions = 4096;                  // layers up to this many positions rank their kept rows in the conv kernel (16 per thread of a 256-thread workgroup)
constexpr int kSplitGrid = 512;                          // workgroups launched when split-K may run
constexpr size_t kSplitTileFloats = 128 * 128;           // largest tile
static inline bool split_k_possible(const Geom &g)
{
    const int64_t tiles64 = (int64_t)((g.m + 127) / 128) * ((g.c_out + 63) / 64);
    return tiles64 < kSplitGrid; // fewer tiles than workgroups even for the dense row count
}
// Fewest stages (128-byte pieces of one tap's channels) a K-split is left with: a layer with fewer than
// two splits' worth is never split, and its calls need no cleared counters.
constexpr int kMinSplitStages = 8;
constexpr int kMaxSplits = 16;         // most K-splits of one tile
constexpr int kBusySplitStages = 64;   // shortest reduction that is split on a busy chip
// Splits of a reduction of `stages` stages (dealt out in `work` pieces) of each of ntiles tiles on `grid` workgroups, two a CU.
// one_a_cu: no more units than a workgroup a CU, as long as that leaves them few stages: two of a CU slow each other, and every split is
// a tile more to park and to read back.  us, two a CU -> one: 488 -> 248, 3x3, on 8 x 15 x 19 (32 tiles in 9 -> 8 splits) 20.0 -> 16.8, E4M3
// 208 -> 64, 5x5 / 2, on 17 x 32 x 87 (52 in 6 -> 4) 22.5 -> 19.3, 384 -> 128, 3x3, on 3 x 60 x 60 15.7 -> 13.8, 512 -> 512 on 32 x 7 x 7 (56 in 9 -> 4)
// 20.6 -> 17.7; without a mask (104 tiles of 72 stages in 4 -> 2) 21.2 -> 21.8, 1024 -> 64 on 5 x 31 x 40 (50 of 144 in 10 -> 5) 18.5 -> 21.6.
__host__ __device__ static inline int split_k_splits(int ntiles, int grid, int work, int stages, bool one_a_cu = false)
{
    int s = grid / ntiles;
    if (one_a_cu && s > 1) {
        const int half = s >> 1; // = grid / (2 * ntiles)
        if (stages <= 24 * half) s = half;
    }
    s = s < 1 ? 1 : (s > work ? work : s);
    if (s > kMaxSplits) s = kMaxSplits;
    // the exchange of partial tiles costs about as much as twenty stages, so a unit keeps at
    // least kMinSplitStages of them: short reductions are not split at all (a 3x3 layer with
    // 64 input channels: 8.4 us unsplit against 19.3 us split three ways)
    const int cap = stages / kMinSplitStages;
    if (s > cap) s = cap < 1 ? 1 : cap;
    // when the tiles alone already fill more than a quarter of the grid, the exchange also
    // competes with the other tiles' traffic and only long reductions gain (512 channels at
    // 16 x 16, batch 16: 72 stages split three ways 31 -> 26 us, 36 stages 20 -> 28 us)
    if (ntiles * 4 > grid && stages < kBusySplitStages) s = 1;
    return s;
}
constexpr int kSmallSplitWaves = 1024; // a 3x3 layer goes to conv_small with at most this many waves
constexpr uint32_t kOneUnitPerCu = 1u << 31; // flag of a launch: split_k_splits' one_a_cu (decided on the host: as device code it cost 0.2 us)
// May the tiled kernel keep its splits to one unit a CU?  Not where another kernel makes the same sums for the same layer, with the list or
// without it: small 16-bit layers (the rules of conv_small_wanted), and all 1x1 kernels on 64 x 64 tiles.
static inline bool splits_of_its_own(const Geom &g, int in_dtype, int tile_rows)
{
    if (tile_rows > 64 || in_dtype == FC_FP8) return true;
    if (g.kh * g.kw != 9) return g.kh * g.kw != 1;
    const int total = 9 * ((g.c_in + 63) / 64);
    return ((g.m + 31) / 32) * ((g.c_out + 31) / 32) * split_k_splits((g.c_out + 63) / 64, kSplitGrid, total, total) > kSmallSplitWaves;
}
constexpr int kSmallLayerTiles = 64;   // layers with at most this many 128 x 64 tiles use small tiles
// Does the tiled kernel take a reduction as one run of 16-byte pieces, eight a stage whatever tap they belong to, instead of tap by tap in whole
// stages?  Where that leaves at most three quarters of the stages: 9 x 72 channels are 11 stages instead of 18, 9 x 16 are 3 instead of 9.
static inline int reduction_stages(const Geom &g, int in_dtype, bool packed)
{
    const int row = g.c_in * (in_dtype == FC_FP8 ? 1 : 2);
    return packed ? (g.kh * g.kw * row + 127) / 128 : g.kh * g.kw * ((row + 127) / 128);
}
// us, tap by tap or on the shared line -> packed, half kept, list given unless said: 72 -> 200 3x3 / 2 on 3 x 75 x 101, mask only, 12.8 -> 10.1, on 4 x 48 x 60
// 17.2 -> 8.2; 16 -> 64 on 16 x 60 x 80, mask only, 15.6 -> 12.4, 5x5 29.5 -> 20.7; 24 -> 128 on 32 x 60 x 80 23.3 -> 17.9, without a mask 32.9 -> 23.9; 72 -> 128 there
// 35.4 -> 32.8, 52.3 -> 47.2; 72 -> 200, 5x5, on 16 x 60 x 80, mask only, 99 -> 70; E4M3 48 -> 80 on 8 x 60 x 80 11.6 -> 9.6.
// On the shared line a stage costs less: where its half-kept tiles are more than one and fewer than two a CU it stays (72 -> 128 on 4 / 6 / 8 / 12 / 20 x 60 x 80 12.8 /
// 13.4 / 14.9 / 17.3 / 23.2 -> 9.9 / 10.5 / 15.9 / 16.1 / 19.5, mask only 15.0 / 15.8 / 18.8 / 21.2 / 27.6 -> 12.9 / 13.6 / 19.2 / 19.7 / 23.0; 136 -> 128 15.7 / 17.0 / 20.6 / 22.7 / 31.5 -> 14.5 /
// 16.3 / 20.8 / 24.1 / 29.7), and without a mask where more than two thirds of the stages are left (136 -> 128 on 8 / 12 x 60 x 80 30.1 / 37.5 -> 30.4 / 40.2).
static inline bool taps_packed(const Geom &g, int in_dtype, bool masked)
{
    const int stages = reduction_stages(g, in_dtype, true), whole = reduction_stages(g, in_dtype, false);
    if (g.kh * g.kw == 1 || 4 * stages > 3 * whole) return false;
    const int64_t tiles64 = (int64_t)((g.m + 127) / 128) * ((g.c_out + 63) / 64);
    const bool line = g.kh == 3 && g.kw == 3 && g.sw == 1 && g.dw == 1 && g.wo >= 32 && g.c_out > 64 && tiles64 >= kSplitGrid;
    return !line || (masked ? tiles64 >= (stages > 16 ? 1000 : 768) : 3 * stages <= 2 * whole);
}
static inline bool split_k_reachable(const Geom &g, int in_dtype, bool masked)
{
    return split_k_possible(g) && reduction_stages(g, in_dtype, taps_packed(g, in_dtype, masked)) >= 2 * kMinSplitStages;
}
static inline size_t split_k_counter_bytes(const Geom &g) { return split_k_possible(g) ? align_up(kSplitGrid * sizeof(int32_t), 256) : 0; }
static inline size_t split_k_partial_bytes(const Geom &g)
{
    return split_k_possible(g) ? (size_t)kSplitGrid * kSplitTileFloats * sizeof(float) : 0;
}
hipError_t launch_zero_i32(int32_t *p, int n, hipStream_t s);

// Matrix-core path (only for shapes conv_mfma_supported accepts).  It also clears
// the irrelevant output rows unless FC_SKIP_ZERO_FILL is set; mask_out may be NULL.
bool tiles_label_rows(const Geom &g, int in_dtype);
// Is the reduction of a layer without a mask split (given split-K scratch)?  Only then are the counters used.  (By the tile that
// launch_conv_mfma takes: both ask choose_tile.)
bool dense_layer_splits(const Geom &g, int in_dtype);
bool conv_mfma_supported(const Geom &g, int in_dtype, int out_dtype);
hipError_t launch_conv_mfma(const Geom &g, int in_dtype, int out_dtype, const void *x,
                            const uint8_t *mask_in, const uint8_t *mask_out, const void *w,
                            const float *bias, const int32_t *idx, const int32_t *count, void *out,
                            float *partials, int32_t *tile_counters, hipStream_t s);

// Layers of a few hundred tiles, 16-bit storage; 1x1 kernels without a list only (see fc_conv_small.hip; shapes
// conv_mfma_supported accepts).  Without a list the kernel labels the positions itself, from mask_out or the
// centre tap of mask_in (needs_labels).  room: partials and tile_counters are there; conv_small_counts: the
// counters are used and must be clear.  as_pw (1x1 kernels): make the sums of launch_conv_pw, in one wave with the bias last.
bool conv_small_wanted(const Geom &g, int in_dtype, bool room, bool needs_labels);
bool conv_small_counts(const Geom &g, bool room);
hipError_t launch_conv_small(const Geom &g, int in_dtype, int out_dtype, bool as_pw, bool room, const void *x, const uint8_t *mask_in,
                             const uint8_t *mask_out, const void *w, const float *bias, const int32_t *idx,
                             const int32_t *count, void *out, float *partials, int32_t *tile_counters, hipStream_t s);

// 3x3 layers of 128-byte pixels with unit horizontal stride and dilation, which launch_conv_pw sends on (see
// fc_conv_res.hip); grid: one workgroup per CU; bias_last: the bias is added to the finished sum, else the sum starts from it.
bool conv_res3_supported(const Geom &g);
// Is the bias of such a layer added last, as on the tap-by-tap form of the resident-weights kernel, or first, as on the
// tiled kernels?  By the sizes each of them served before this kernel, so that a layer keeps its sums: a changed last bit of a few
// 16-bit values is 1 % of the outputs fifty layers on.
bool conv_res3_bias_last(const Geom &g, bool masked);
hipError_t launch_conv_res3(const Geom &g, int in_dtype, int out_dtype, int grid, bool bias_last, const void *x, const uint8_t *mask_in,
                            const uint8_t *mask_out, const void *w, const float *bias, const int32_t *idx, const int32_t *count,
                            void *out, hipStream_t s);

// 3x3 layers with several wide tiles per CU (see fc_conv_wide.hip; shapes conv_mfma_supported accepts): whole chunks of
// input channels, whole 128-channel blocks of output channels, unit horizontal stride and dilation.  Needs the kept list (or
// no mask at all); grid: one workgroup per CU.
bool conv_wide_supported(const Geom &g, int in_dtype, int out_dtype);
hipError_t launch_conv_wide(const Geom &g, int in_dtype, int out_dtype, int grid, const void *x, const uint8_t *mask_in,
                            const uint8_t *mask_out, const void *w, const float *bias, const int32_t *idx, const int32_t *count,
                            void *out, hipStream_t s);
int conv_grid_cus(); // the CU count, a multiple of the XCD count (read once per process; all devices of a node are alike)

// Calibration launches (see fc_calibrate.hip): `blocks` workgroups of four waves each run
// `iters` rounds of eight matrix instructions; a streaming copy of `bytes` bytes.
hipError_t launch_calibrate_mfma(int dtype, int iters, int blocks, float *sink, hipStream_t s);
hipError_t launch_calibrate_copy(const void *src, void *dst, size_t bytes, hipStream_t s);
// `steps` steps of two matrix instructions plus item `mode` per wave, 1, 2 or 4 waves per SIMD;
// cycles[block] = shader cycles of the loop.
hipError_t launch_calibrate_issue(int mode, int waves_per_simd, int steps, int blocks, const void *src,
                                  long long *cycles, float *sink, hipStream_t s);

// One-workgroup-per-CU matrix-core path for 3x3 layers (see fc_conv_line.hip): 128 output
// channels per tile.  Needs the kept list (or no mask at all).
bool conv_line_supported(const Geom &g, int in_dtype, int out_dtype);
hipError_t launch_conv_line(const Geom &g, int in_dtype, int out_dtype, const void *x,
                            const uint8_t *mask_in, const uint8_t *mask_out, const void *w, const float *bias,
                            const int32_t *idx, const int32_t *count, void *out, hipStream_t s);

// Resident-weights matrix-core path (see fc_conv_pw.hip): 1x1 layers without padding whose rows
// are whole 16-byte pieces and whose weights, cut into slices of output channels, stay in LDS,
// and 3x3 layers whose pixels are 128 bytes (bf16, f16 or E4M3 storage).  Needs the kept list
// (or no mask at all).
bool conv_pw_supported(const Geom &g, int in_dtype, int out_dtype);
hipError_t launch_conv_pw(const Geom &g, int in_dtype, int out_dtype, const void *x, const uint8_t *mask_in,
                          const uint8_t *mask_out, const void *w, const float *bias, const int32_t *idx,
                          const int32_t *count, void *out, hipStream_t s);

// Two 1x1 layers, the second the only reader of the first, in one launch (see fc_conv_pair.hip): unit stride, the same kept
// rows, storage of one type throughout, irrelevant rows of the output left alone.  bias_first: the layer's sum starts from its
// bias, as on the tiled kernels, else the bias is added to the finished sum, as on the resident-weights kernel.
bool conv_pair_supported(const Geom &g1, const Geom &g2, int dtype);
hipError_t launch_conv_pair(const Geom &g1, const Geom &g2, int dtype, bool bias_first1, bool bias_first2, const void *x, const void *w1,
                            const float *bias1, const void *w2, const float *bias2, const int32_t *idx, const int32_t *count, void *out,
                            hipStream_t s);

} // namespace fc
