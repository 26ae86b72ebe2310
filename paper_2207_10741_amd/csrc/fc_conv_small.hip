// Focused convolution on the matrix cores for layers of a few hundred row blocks (the layers of a
// network at batch 1 to 4; 16-bit storage; 1x1 kernels where no list is given).
//
// Such a layer is a chain of memory round trips: its matrix work takes a tenth of its time.  This
// kernel is cut for the chain, not for the throughput:
//   - a wave owns 32 rows x 32 channels and, where the reduction is long, one split of it; the splits of a
//     tile are the waves of one workgroup (of several, past four) and meet in LDS.  Splits and the order
//     within them are those of the tiled kernel: the same sums, bit for bit;
//   - every wave is a pipeline of its own: it stages its own pixels and weights in its own ring of LDS
//     slots (a slot = 64 channels of one tap for the tile's rows and channels), with no barrier
//     before the sums of the waves meet;
//   - the tile of a workgroup follows from its number alone, so the weights of its first slots are
//     requested before anything is known about its rows;
//   - with a list, the count travels while the weights are requested, then the entries below it are read;
//     without one, a tile is 32 consecutive positions, labelled here: no compaction before the
//     kernel and no zero-fill after it, irrelevant rows come out as zeros;
//   - pixels are gathered as soon as their addresses are known; what the input mask says about
//     them arrives meanwhile and is applied to the operand as it is read from LDS.
// (3x3 layers whose waves have at most nine stages run on k_conv_small_once, below.)
// (The tiled kernel took 17 000 cycles for 64 -> 64 at 56 x 56: 1 400 for the count, 4 300 to the rows'
// addresses, 2 000 for the tap bits, 6 100 for nine stages of which 1 150 are matrix instructions.)
#include "fc_dma_util.hpp"
#include <type_traits>
#include <atomic>

namespace fc {

constexpr int kSmallRows = 32, kSmallChannels = 32;
constexpr int kSmallSlots = 4;
constexpr int kSmallWaves = 4;      // most waves of a workgroup
constexpr uint32_t kSmallSlotBytes = (kSmallRows + kSmallChannels) * 128u;
constexpr uint32_t kSmallWaveBytes = kSmallSlots * kSmallSlotBytes;

// How the launch is cut: channel tiles, groups of (up to four) splits, and the divisions of the workgroup number.
struct SmallCut {
    int32_t n_nt, groups, room;
    int32_t splits;    // where they do not depend on the kept count
    FastDiv per_mt;    // by n_nt * groups
    FastDiv by_groups;
    FastDiv by_cch;    // by the 64-channel chunks of a tap
    FastDiv by_kw;
    FastDiv by_splits;
};

// Splits of every tile's reduction when `rows` rows are kept: for 3x3 and 1x1 kernels the tiled kernel's rule for its
// 64 x 64 tiles (which splits nothing without a workspace: 384 -> 48 on 4 x 26 x 14, 54 stages in one wave, 22.0 us, in
// four 9.8 us); the others never ran there on such tiles and are cut for the waves of one workgroup.
__host__ __device__ static inline int small_splits(int rows, int c_out, int stages, int taps, bool room)
{
    if ((taps | 8) != 9) return stages >= 4 * kSmallWaves ? kSmallWaves : 1;
    const int ntiles = ((rows + 63) / 64) * ((c_out + 63) / 64);
    if (!room) { // no workspace to meet in: the waves of a workgroup
        const int cap = stages / kMinSplitStages;
        return cap < 1 ? 1 : (cap < kSmallWaves ? cap : kSmallWaves);
    }
    return ntiles > 0 ? split_k_splits(ntiles, kSplitGrid, stages, stages) : 1;
}

// What a wave of a tile knows when its products are done.
struct SmallUnit {
    int waves, wave;          // of the workgroup
    int mt, nt, group;        // row tile, channel tile, group of splits
    int splits, split;        // of the tile, this wave's
    int co0, r0;              // first channel and row
    int p;                    // position of this lane's row
    bool live, drop;          // the row is kept; it is an irrelevant position
};

// The sums of a tile meet in LDS (past the waves of one workgroup through the workspace), in split order, and are stored.
template <int DT, typename TO>
__device__ __forceinline__ void small_meet_and_store(const Geom &g, const SmallUnit &u, int n_nt, bool fill, const f32x16_t &acc, unsigned char *lds,
                                                     TO *__restrict__ out, float *__restrict__ partials, int32_t *__restrict__ tile_counters)
{
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const bool mine = u.live || (u.drop && fill);
    const int64_t orow = (g.flags & FC_COMPACT_OUT) ? (int64_t)u.r0 + l32 : (int64_t)(u.drop ? u.r0 + l32 : u.p);
    TO *const to = out + orow * g.c_out + (u.co0 + half * 4);
    // quad q of a lane = channels 8 q + 4 half .. + 3 of its row; wave v finishes quads v, v + waves, ...
    auto store = [&](int q, const float4 &t_in) __attribute__((always_inline)) {
        const int co = u.co0 + q * 8 + half * 4;
        if (co >= g.c_out || !mine) return;
        float4 t = u.drop ? make_float4(0.f, 0.f, 0.f, 0.f) : t_in;
        TO *o = to + q * 8;
        if constexpr (sizeof(TO) == 4) {
            if (g.flags & FC_RELU) {
                t.x = relu_keep_nan(t.x); t.y = relu_keep_nan(t.y);
                t.z = relu_keep_nan(t.z); t.w = relu_keep_nan(t.w);
            }
            store4<DT, TO>(o, t.x, t.y, t.z, t.w);
        } else if constexpr (sizeof(TO) == 1) {
            uint32_t pk;
            store4<DT, TO>(reinterpret_cast<TO *>(&pk), t.x, t.y, t.z, t.w);
            if (g.flags & FC_RELU) pk = relu_packed8(pk);
            *reinterpret_cast<uint32_t *>(o) = pk;
        } else {
            uint2 pk;
            store4<DT, TO>(reinterpret_cast<TO *>(&pk), t.x, t.y, t.z, t.w);
            if (g.flags & FC_RELU) {
                pk.x = relu_packed16(pk.x);
                pk.y = relu_packed16(pk.y);
            }
            *reinterpret_cast<uint2 *>(o) = pk;
        }
    };
    const int mates = (u.splits + u.waves - 1) / u.waves; // workgroups that share the tile
    if (u.splits == 1) {
        if (u.wave == 0 && u.group == 0)
#pragma unroll
            for (int q = 0; q < 4; ++q) store(q, make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]));
    } else if (mates == 1) {
        if (u.group == 0) { // uniform
            __syncthreads(); // every u.wave is done with its slots
            float4 *part = reinterpret_cast<float4 *>(lds);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                part[(u.wave * 4 + q) * 64 + lane] = make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
            __syncthreads();
            for (int q = u.wave; q < 4; q += u.waves) {
                float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
                for (int k = 0; k < u.splits; ++k) {
                    const float4 t = part[(k * 4 + q) * 64 + lane];
                    v.x += t.x; v.y += t.y; v.z += t.z; v.w += t.w;
                }
                store(q, v);
            }
        }
    } else if (u.group < mates) { // uniform
        // Park the sums (device-scope accesses, as in the tiled kernel), count in; the workgroup that
        // arrives last adds the partial tiles in u.split order.
        const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(
            partials, 0, (uint32_t)((size_t)kSplitGrid * kSplitTileFloats * sizeof(float)), 0x00020000);
        constexpr uint32_t TILE = (uint32_t)kSmallRows * kSmallChannels * 4u;
        const int tile = u.mt * n_nt + u.nt;
        const uint32_t first = (uint32_t)(tile * u.splits) * TILE;
        if (u.split < u.splits)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                u32x4_t t;
                t.x = __float_as_uint(acc[4 * q]); t.y = __float_as_uint(acc[4 * q + 1]);
                t.z = __float_as_uint(acc[4 * q + 2]); t.w = __float_as_uint(acc[4 * q + 3]);
                __builtin_amdgcn_raw_buffer_store_b128(t, rp, first + (uint32_t)u.split * TILE + (uint32_t)(q * 64 + lane) * 16u,
                                                       0, kDeviceScope);
            }
        wait_vmcnt<0>();
        __syncthreads();
        int *arrived = reinterpret_cast<int *>(lds);
        if (tid == 0)
            *arrived = __hip_atomic_fetch_add(&tile_counters[tile], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (*arrived == mates - 1) {
            if (tid == 0) // leave the counters as they were found
                __hip_atomic_store(&tile_counters[tile], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            for (int q = u.wave; q < 4; q += u.waves) {
                u32x4_t t[kMaxSplits]; // all partial tiles in flight
#pragma unroll
                for (int k = 0; k < kMaxSplits; ++k)
                    t[k] = __builtin_amdgcn_raw_buffer_load_b128(
                        rp, k < u.splits ? first + (uint32_t)k * TILE + (uint32_t)(q * 64 + lane) * 16u : kOutOfRange, 0, kDeviceScope);
                float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                for (int k = 0; k < kMaxSplits; ++k) { // (zeros past the last u.split)
                    v.x += __uint_as_float(t[k].x); v.y += __uint_as_float(t[k].y);
                    v.z += __uint_as_float(t[k].z); v.w += __uint_as_float(t[k].w);
                }
                store(q, v);
            }
        }
    }
}

// 32 irrelevant positions in a row
template <typename TO>
__device__ __forceinline__ void small_clear_tile(const Geom &g, const SmallUnit &u, TO *__restrict__ out)
{
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const int pieces = min(kSmallChannels, g.c_out - u.co0) * (int)sizeof(TO) / 16;
    const u32x4_t zero = {0u, 0u, 0u, 0u};
    for (int i = u.wave * 2 + half; i < pieces; i += 2 * u.waves)
        *reinterpret_cast<u32x4_t *>(out + (int64_t)(u.r0 + l32) * g.c_out + u.co0 + i * (16 / (int)sizeof(TO))) = zero;
}

// With a list: the irrelevant rows, by the workgroups whose tile does not exist when there are enough.  Every wave has waited for its own
// loads; the waves' lists lie in the first wave's slots, where its weights and pixels (in k_conv_small_once the weights of idle tiles too) and the sums of
// a tile come to lie, so all waves meet before the first entry is written.
template <typename TO>
__device__ __forceinline__ void small_clear_rest(const Geom &g, const SmallUnit &u, int tiles, int nts, const uint8_t *__restrict__ mask_in,
                                                 const uint8_t *__restrict__ mask_out, TO *__restrict__ out, unsigned char *lds)
{
    const int unit = blockIdx.x, grid = gridDim.x, idle = grid - tiles * nts;
    const bool idle_only = idle * 16 >= grid;
    if (!idle_only || u.mt >= tiles) {
        __syncthreads(); // (the condition is the workgroup's)
        clear_irrelevant(g, mask_in, mask_out, out, g.c_out * (int)sizeof(TO) / 16,
                         (idle_only ? unit - tiles * nts : unit) * u.waves + u.wave, (idle_only ? idle : grid) * u.waves,
                         reinterpret_cast<int32_t *>(lds) + u.wave * 64);
    }
}

// BIAS_LAST (1x1 kernels): the bias is added to the finished sums instead of starting them.  (An instance of its own: chosen at run time, by a
// select an accumulator, it cost 0.2 to 0.4 us of the 4.8 of a 1x1 layer, 0.7 of the 7.9 of a 3x3 one.)
template <int DT, typename TO, bool BIAS_LAST>
__global__ __launch_bounds__(64 * kSmallWaves, 1) void k_conv_small(Geom g, SmallCut cut, const uint16_t *__restrict__ x,
                                                                 const uint8_t *__restrict__ mask_in,
                                                                 const uint8_t *__restrict__ mask_out,
                                                                 const uint16_t *__restrict__ w,
                                                                 const float *__restrict__ bias,
                                                                 const int32_t *__restrict__ idx,
                                                                 const int32_t *__restrict__ count, TO *__restrict__ out,
                                                                 float *__restrict__ partials,
                                                                 int32_t *__restrict__ tile_counters)
{
    constexpr int NS = kSmallSlots;
    constexpr int XL = kSmallRows / 8, WL = kSmallChannels / 8; // wave loads of a slot: 8 rows of 128 bytes each
    constexpr uint32_t SLOT = kSmallSlotBytes;
    extern __shared__ __align__(16) unsigned char lds[];

    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int waves = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int unit = blockIdx.x, nts = cut.n_nt * cut.groups;
    const int mt = (int)fast_div((uint32_t)unit, cut.per_mt), in_mt = unit - mt * nts;
    const int nt = (int)fast_div((uint32_t)in_mt, cut.by_groups), group = in_mt - nt * cut.groups;
    const int co0 = nt * kSmallChannels, r0 = mt * kSmallRows;
    const int taps = g.kh * g.kw, cch = (g.c_in + 63) >> 6, total = taps * cch;
    const int split = group * waves + wave;
    // this wave's stages [q0, q0 + n)
    int rows = g.m, splits = 1, q0 = 0, n = 0;
    auto take_split = [&]() {
        splits = small_splits(rows, g.c_out, total, taps, cut.room != 0);
        const uint32_t b = splits > 1 ? (uint32_t)(split * total) / (uint32_t)splits : 0u;
        const uint32_t e = splits > 1 ? (uint32_t)((split + 1) * total) / (uint32_t)splits : (uint32_t)total;
        q0 = (int)b;
        n = split < splits ? (int)(e - b) : 0;
    };
    // (with a list the splits follow the kept count; when that could change them, the count is waited for)
    const bool wait_count = idx && small_splits(1, g.c_out, total, taps, cut.room != 0) != small_splits(g.m, g.c_out, total, taps, cut.room != 0);
    const int listed = idx ? *count : 0;
    if (wait_count) rows = listed;
    take_split();

    const uint32_t lds_wave = __builtin_amdgcn_readfirstlane((uint32_t)reinterpret_cast<uintptr_t>(lds) + (uint32_t)wave * kSmallWaveBytes);
    const unsigned char *my_lds = lds + (uint32_t)wave * kSmallWaveBytes;
    const int prow = lane >> 3;
    // (rows of a lane's loads differ by multiples of 8: the swizzle alternates with bit 2 of (row >> 1))
    const int piece0 = (lane & 7) ^ FC_SWZ(prow), piece1 = (lane & 7) ^ FC_SWZ(prow + 8);

    // ---- weights of the first slots ----
    const u32x4_t rsrc_w = make_rsrc_words(w, (uint32_t)g.c_out * taps * g.c_in * 2u);
    // (Code that runs once is kept short - loops rolled - since fetching it is what it costs; the loop over
    // the stages steps its cursors instead of dividing.)
    struct Cursor {
        int tap, cc, kh, kw, left; // left: stages to come
    };
    auto cursor_at = [&](int q, int left) {
        Cursor c;
        c.tap = (int)fast_div((uint32_t)q, cut.by_cch);
        c.cc = q - c.tap * cch;
        c.kh = (int)fast_div((uint32_t)c.tap, cut.by_kw);
        c.kw = c.tap - c.kh * g.kw;
        c.left = left;
        return c;
    };
    auto advance = [&](Cursor &c) {
        --c.left;
        if (++c.cc == cch) {
            c.cc = 0;
            ++c.tap;
            if (++c.kw == g.kw) {
                c.kw = 0;
                ++c.kh;
            }
        }
    };
    const int ch0 = piece0 * 8, ch1 = piece1 * 8;
    // weight rows past the last channel lie past the tensor's end and read as zeros
    uint32_t woff[WL];
#pragma unroll
    for (int j = 0; j < WL; ++j)
        woff[j] = (uint32_t)(co0 + prow + 8 * j) * (uint32_t)(taps * g.c_in) * 2u + (uint32_t)(j & 1 ? ch1 : ch0) * 2u;
    auto load_w = [&](const Cursor &c, int slot) __attribute__((always_inline)) {
        uint32_t sw = (uint32_t)(c.tap * g.c_in + c.cc * 64) * 2u;
        sw = __builtin_amdgcn_readfirstlane(c.left > 0 ? sw : 0u);
        __asm__("" : "+s"(sw));
        const int room = c.left > 0 ? g.c_in - c.cc * 64 : 0;
        const uint32_t to = lds_wave + (uint32_t)slot * SLOT + (uint32_t)kSmallRows * 128u;
#pragma unroll
        for (int j = 0; j < WL; ++j)
            dma_load16_s(rsrc_w, (j & 1 ? ch1 : ch0) < room ? woff[j] : kOutOfRange, sw,
                         __builtin_amdgcn_readfirstlane(to + (uint32_t)j * 1024u));
    };
    Cursor wc = cursor_at(q0, n);
#pragma unroll 1
    for (int i = 0; i < NS - 1; ++i) {
        load_w(wc, i);
        advance(wc);
    }

    // ---- the tile's rows: lane l holds row l & 31 ----
    const bool packed = (g.flags & FC_PACKED_MASKS) != 0;
    const bool fill = mask_in && !(g.flags & FC_SKIP_ZERO_FILL);
    int p = r0 + l32;
    bool live = p < g.m, drop = false;
    if (idx) {
        // (entries past the count are not read: a caller's list may end there)
        rows = listed;
        live = p < rows;
        p = live ? idx[p] : 0;
    } else if (mask_in) {
        const bool kept = live && position_kept(g, mask_in, mask_out, live ? p : 0);
        drop = live && !kept;
        live = kept;
    }
    const int tiles = (rows + kSmallRows - 1) / kSmallRows; // row tiles that exist
    const bool any = __ballot(live) != 0;
    if (any) {
        const int q = (int)fast_div((uint32_t)(live ? p : 0), g.div_wo), ow = (live ? p : 0) - q * g.wo;
        const int img = (int)fast_div((uint32_t)q, g.div_ho), oh = q - img * g.ho;
        const int ih0 = oh * g.sh - g.ph, iw0 = ow * g.sw - g.pw;
        const int pix0 = (img * g.h + ih0) * g.w + iw0; // may lie outside the image
        // taps inside the image
        uint32_t inside = 0;
        if (live) {
            uint32_t cols = 0;
            for (int k = 0; k < g.kw; ++k) cols |= (uint32_t)(iw0 + k * g.dw) < (uint32_t)g.w ? 1u << k : 0u;
            for (int k = 0; k < g.kh; ++k)
                if ((uint32_t)(ih0 + k * g.dh) < (uint32_t)g.h) inside |= cols << (k * g.kw);
        }
        // pixels are read through a descriptor that starts a padding's worth before the tensor, so that no
        // offset is negative (taps outside the image are switched off)
        const uint32_t xbias = (uint32_t)(g.ph * g.w + g.pw) * (uint32_t)g.c_in * 2u;
        const u32x4_t rsrc_x = make_rsrc_words(reinterpret_cast<const unsigned char *>(x) - xbias,
                                               (uint32_t)g.n * g.h * g.w * g.c_in * 2u + xbias);
        uint32_t xoff[XL], xin[XL];
#pragma unroll
        for (int j = 0; j < XL; ++j) {
            const int r = prow + 8 * j;
            xoff[j] = (uint32_t)__shfl(pix0, r) * (uint32_t)g.c_in * 2u + xbias + (uint32_t)((j & 1 ? piece1 : piece0) * 16);
            xin[j] = (uint32_t)__shfl((int)inside, r);
        }
        auto load_x = [&](const Cursor &c, int slot) __attribute__((always_inline)) {
            uint32_t sx = (uint32_t)((c.kh * g.dh * g.w + c.kw * g.dw) * g.c_in + c.cc * 64) * 2u;
            sx = __builtin_amdgcn_readfirstlane(c.left > 0 ? sx : 0u);
            __asm__("" : "+s"(sx));
            const int room = c.left > 0 ? g.c_in - c.cc * 64 : 0;
            const uint32_t bit = 1u << (c.tap & 31);
            const uint32_t sel0 = ch0 < room ? bit : 0u, sel1 = ch1 < room ? bit : 0u;
            const uint32_t to = lds_wave + (uint32_t)slot * SLOT;
#pragma unroll
            for (int j = 0; j < XL; ++j)
                dma_load16_s(rsrc_x, (xin[j] & (j & 1 ? sel1 : sel0)) ? xoff[j] : kOutOfRange, sx,
                             __builtin_amdgcn_readfirstlane(to + (uint32_t)j * 1024u));
        };
        Cursor xc = cursor_at(q0, n);
#pragma unroll 1
        for (int i = 0; i < NS - 1; ++i) {
            load_x(xc, i);
            advance(xc);
        }

        // what the mask says about this lane's row under the wave's taps
        uint32_t bits = inside;
        if (mask_in) {
            const int t0 = cursor_at(q0, 0).tap, t1 = cursor_at(n > 0 ? q0 + n - 1 : q0, 0).tap;
            const int64_t mask_bytes = (int64_t)g.n * g.h * g.w;
            uint32_t rel = 0;
            if (!packed && g.dw == 1 && g.kw <= 4 && mask_bytes >= 4) {
                // the taps of a kernel row with one (unaligned) 4-byte load; one that would leave the mask is
                // moved inside it and its bytes moved back
                const int k0 = (int)fast_div((uint32_t)t0, cut.by_kw), k1 = (int)fast_div((uint32_t)t1, cut.by_kw);
                constexpr int U = 3;
#pragma unroll 1
                for (int k = k0; k <= k1; k += U) {
                    uint32_t m[U];
                    int moved[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int off = live && k + u <= k1 ? pix0 + (k + u) * g.dh * g.w : 0; // (positions fit 31 bits)
                        const int at = min(max(off, 0), (int)mask_bytes - 4);
                        moved[u] = off - at;
                        __builtin_memcpy(&m[u], mask_in + at, 4);
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        uint32_t v = moved[u] < 0 ? (moved[u] > -4 ? m[u] << (-8 * moved[u]) : 0u)
                                                  : (moved[u] < 4 ? m[u] >> (8 * moved[u]) : 0u);
                        v = (((v & 0x7f7f7f7fu) + 0x7f7f7f7fu) | v) & 0x80808080u; // nonzero bytes
                        v = ((v >> 7) & 1u) | ((v >> 14) & 2u) | ((v >> 21) & 4u) | (v >> 28);
                        if (k + u <= k1) rel |= (v & ((1u << g.kw) - 1u)) << ((k + u) * g.kw);
                    }
                }
            } else {
#pragma unroll 1
                for (int t = t0; t <= t1; ++t) {
                    const int kh = (int)fast_div((uint32_t)t, cut.by_kw), kw = t - kh * g.kw;
                    const bool in = (inside >> t) & 1u;
                    if (mask_at(mask_in, in ? pix0 + kh * g.dh * g.w + kw * g.dw : 0, packed)) rel |= 1u << t;
                }
            }
            bits &= rel;
        }

        // the sums start from the bias (first split)
        f32x16_t acc;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int co = co0 + q * 8 + half * 4;
            float4 bq = make_float4(0.f, 0.f, 0.f, 0.f);
            if (bias && split == 0 && co < g.c_out) bq = *reinterpret_cast<const float4 *>(bias + co);
            acc[4 * q] = bq.x; acc[4 * q + 1] = bq.y; acc[4 * q + 2] = bq.z; acc[4 * q + 3] = bq.w;
        }
        f32x16_t last;
        if constexpr (BIAS_LAST) {
            last = acc;
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[i] = 0.f;
        }
        const uint32_t frag = (uint32_t)l32 * 128u, swz = FC_SWZ(l32);
        // A step multiplies the operands it finds in registers, after requesting the next stage's from LDS;
        // the slot they came from is then free and takes the stage NS - 1 further on.
        struct Operands {
            Frag<DT> x[4], w[4];
        };
        auto fetch = [&](Operands &o, int slot) __attribute__((always_inline)) {
            const unsigned char *xs = my_lds + (uint32_t)slot * SLOT + frag, *ws = xs + kSmallRows * 128;
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                const uint32_t at = (uint32_t)((2 * kk + half) ^ swz) * 16u;
                o.x[kk].load(xs, at);
                o.w[kk].load(ws, at);
            }
        };
        Cursor mc = cursor_at(q0, n);
        int slot = 0; // of the stage about to be multiplied
        auto step = [&](Operands &now, Operands &next) __attribute__((always_inline)) {
            const int after = slot + 1 == NS ? 0 : slot + 1;
            wait_vmcnt<(XL + WL) * (NS - 3)>(); // the next stage has landed
            fetch(next, after);
            __builtin_amdgcn_sched_barrier(0);
            const int last = slot == 0 ? NS - 1 : slot - 1; // (free since the step before)
            load_w(wc, last);
            load_x(xc, last);
            advance(wc);
            advance(xc);
            const bool on = (bits >> (mc.tap & 31)) & 1u;
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                now.x[kk].v.x = on ? now.x[kk].v.x : 0u;
                now.x[kk].v.y = on ? now.x[kk].v.y : 0u;
                now.x[kk].v.z = on ? now.x[kk].v.z : 0u;
                now.x[kk].v.w = on ? now.x[kk].v.w : 0u;
                acc = mfma32<DT>(now.w[kk], now.x[kk], acc);
            }
            advance(mc);
            slot = after;
            // (operands read before their slot is written again: the loads above go to the slot of the
            // step before, whose operands have been multiplied)
        };
        Operands oa, ob;
        wait_vmcnt<0>(); // the first NS - 1 slots
        fetch(oa, 0);
#pragma unroll 1
        for (int i = 0; i < n; i += 2) {
            step(oa, ob);
            if (i + 1 >= n) break;
            step(ob, oa);
        }
        wait_vmcnt<0>();
        if constexpr (BIAS_LAST)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[i] += last[i];

        const SmallUnit u = {waves, wave, mt, nt, group, splits, split, co0, r0, p, live, drop};
        small_meet_and_store<DT, TO>(g, u, cut.n_nt, fill, acc, lds, out, partials, tile_counters);
    } else {
        wait_vmcnt<0>(); // (weights on their way into LDS)
        if (fill && drop && group == 0) {
            const SmallUnit u = {waves, wave, mt, nt, group, splits, split, co0, r0, p, live, drop};
            small_clear_tile(g, u, out);
        }
    }
    if (idx && fill) {
        const SmallUnit u = {waves, wave, mt, nt, group, splits, split, co0, r0, p, live, drop};
        small_clear_rest(g, u, tiles, nts, mask_in, mask_out, out, lds);
    }
}

// 3x3 layers of whole 64-channel chunks whose waves have eight or nine stages each: everything on its way at once.  A wave that has a
// SIMD to itself issues an instruction every four to five cycles, whatever it is, and a 1 KB load into LDS every 25; the loops of the
// kernel above came to 60 cycles a load of weights, 106 a load of pixels and 395 a stage (stamps, 64 -> 64 on 56 x 56: 15 600 cycles, of
// which matrix instructions 1 150).  Here nothing is computed per load that a layer of this kind does not need:
//   - what decides about the rows (labels or list entries) is requested before the weights;
//   - the weights of all stages pass through LDS into registers while the rows' addresses are computed; the pixels then take their place;
//   - a pixel's offset is one addition: what lies outside the tensor is out of the descriptor's range, what lies in it beside the image
//     is dropped with the irrelevant pixels, by reading a row of zeros instead;
//   - the stages are straight-line code (a branch into code not fetched yet costs 500 cycles), so waits and LDS offsets are constants.
// The products and their order are those of the kernel above.  One launch after another, half kept, us, kernel above -> here: 64 -> 64 on 56 x 56
// 7.5 -> 4.4 (8 250 cycles: 2 200 to the last load of weights, 2 800 to the last of pixels, 2 300 in the stages), 128 -> 128 on 28 x 28 8.0 -> 5.0,
// 256 -> 256 on 14 x 14 8.3 -> 6.0, 512 -> 512 on 7 x 7 9.4 -> 7.5 (four waves of a CU: 288 KB through its L1 at 22 cycles a KB).
constexpr int kOnceStages = 9; // (a wave of eight leaves the first one out)
constexpr uint32_t kOnceSlot = kSmallRows * 128u;
constexpr uint32_t kOnceZeros = kOnceStages * kOnceSlot;
constexpr uint32_t kOnceWaveBytes = kOnceZeros + 128u;
static_assert(kSmallRows == kSmallChannels, "pixels take the place of the weights");

// A 1 KB load into LDS at base + at (a constant once inlined).
__device__ __forceinline__ void once_load(const u32x4_t &rsrc, uint32_t byte_offset, uint32_t scalar_offset, uint32_t base, uint32_t at)
{
    __asm__ volatile("s_add_u32 m0, %0, %4\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                     :
                     : "s"(base), "v"(byte_offset), "s"(rsrc), "s"(scalar_offset), "n"(at)
                     : "memory", "scc");
}

template <int DT, typename TO>
__global__ __launch_bounds__(64 * kSmallWaves, 1) void k_conv_small_once(Geom g, SmallCut cut, const uint16_t *__restrict__ x,
                                                                      const uint8_t *__restrict__ mask_in,
                                                                      const uint8_t *__restrict__ mask_out,
                                                                      const uint16_t *__restrict__ w,
                                                                      const float *__restrict__ bias,
                                                                      const int32_t *__restrict__ idx,
                                                                      const int32_t *__restrict__ count, TO *__restrict__ out,
                                                                      float *__restrict__ partials,
                                                                      int32_t *__restrict__ tile_counters)
{
    constexpr int ST = kOnceStages;
    extern __shared__ __align__(16) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int waves = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int unit = blockIdx.x, nts = cut.n_nt * cut.groups;
    const int mt = (int)fast_div((uint32_t)unit, cut.per_mt), in_mt = unit - mt * nts;
    const int nt = (int)fast_div((uint32_t)in_mt, cut.by_groups), group = in_mt - nt * cut.groups;
    const int co0 = nt * kSmallChannels, r0 = mt * kSmallRows;
    const int split = group * waves + wave, cch = g.c_in >> 6, splits = cut.splits;
    const bool fill = mask_in && !(g.flags & FC_SKIP_ZERO_FILL);
    // this wave's stages: q0 .. q0 + n - 1 (waves past the last split: none)
    const bool busy = split < splits;
    const int q0 = busy ? (int)fast_div((uint32_t)(split * 9 * cch), cut.by_splits) : 0;
    const bool skip = (int)fast_div((uint32_t)((split + 1) * 9 * cch), cut.by_splits) - q0 < ST; // the first of the nine is left out

    // ---- request what decides about the rows: lane l holds row l & 31 ----
    const int rows = idx ? __builtin_amdgcn_readfirstlane(*count) : g.m;
    int p = r0 + l32;
    bool live = p < rows;
    // (values of loads that are waited for by hand are touched by nothing before the wait)
    uint32_t entry, label;
    if (idx) {
        // (entries past the count are not read: a caller's list may end there)
        const u32x4_t rsrc_i = make_rsrc_words(idx, (uint32_t)rows * 4u);
        __asm__ volatile("buffer_load_dword %0, %1, %2, 0 offen" : "=v"(entry) : "v"((uint32_t)p * 4u), "s"(rsrc_i) : "memory");
    } else if (mask_in) {
        int at = live ? p : 0;
        if (!mask_out) { // under the centre tap
            const int q = (int)fast_div((uint32_t)at, g.div_wo), ow = at - q * g.wo;
            const int img = (int)fast_div((uint32_t)q, g.div_ho), oh = q - img * g.ho;
            const int ih = min(max(oh * g.sh - g.ph + g.dh, 0), g.h - 1), iw = min(max(ow * g.sw - g.pw + 1, 0), g.w - 1);
            at = (img * g.h + ih) * g.w + iw;
        }
        __asm__ volatile("global_load_ubyte %0, %1, %2" : "=v"(label) : "v"(at), "s"(mask_out ? mask_out : mask_in) : "memory");
    }
    // the sums start from the bias (first split)
    const u32x4_t rsrc_b = make_rsrc_words(bias, bias && split == 0 ? (uint32_t)g.c_out * 4u : 0u);
    u32x4_t bq[4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
        __asm__ volatile("buffer_load_dwordx4 %0, %1, %2, 0 offen" : "=v"(bq[r]) : "v"((uint32_t)(co0 + r * 8 + half * 4) * 4u), "s"(rsrc_b) : "memory");

    // ---- weights of all stages ----
    const uint32_t lds_wave = __builtin_amdgcn_readfirstlane((uint32_t)reinterpret_cast<uintptr_t>(lds) + (uint32_t)wave * kOnceWaveBytes);
    unsigned char *my_lds = lds + (uint32_t)wave * kOnceWaveBytes;
    const int prow = lane >> 3;
    // (rows of a lane's loads differ by multiples of 8: the swizzle alternates with bit 2 of (row >> 1))
    const uint32_t piece0 = (uint32_t)((lane & 7) ^ FC_SWZ(prow)) * 16u, piece1 = (uint32_t)((lane & 7) ^ FC_SWZ(prow + 8)) * 16u;
    const uint32_t pixel = (uint32_t)g.c_in * 2u, wrow = 9u * pixel;
    const u32x4_t rsrc_w = make_rsrc_words(w, (uint32_t)g.c_out * wrow);
    uint32_t woff[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int co = co0 + prow + 8 * j;
        uint32_t off = (uint32_t)co * wrow + (j & 1 ? piece1 : piece0);
        __asm__("" : "+v"(off));
        woff[j] = co < g.c_out && busy ? off : kOutOfRange;
    }
    // Lane e < 9 knows stage e: its channels' offset in a weight row, its pixels' offset from those of tap 0, and its tap.  (Where the
    // first stage is left out, its place holds what the second one's does.)
    const int q_e = q0 + min(max(lane - (skip ? 1 : 0), 0), ST - 1);
    const int tap_e = (int)fast_div((uint32_t)q_e, cut.by_cch), kh_e = tap_e * 11 >> 5;
    const int w_e = q_e * 128, x_e = (kh_e * g.dh * g.w + (tap_e - 3 * kh_e)) * (int)pixel + (q_e - tap_e * cch) * 128, bit_e = 1 << tap_e;
    uint32_t sw[ST]; // (all before the first load: a scalar register that the vector unit wrote may not be read by a load right after)
#pragma unroll
    for (int e = 0; e < ST; ++e) {
        sw[e] = (uint32_t)__builtin_amdgcn_readlane(w_e, e);
        __asm__ volatile("" : "+s"(sw[e]));
    }
    __asm__ volatile("s_nop 4");
#pragma unroll
    for (int e = 0; e < ST; ++e)
#pragma unroll
        for (int j = 0; j < 4; ++j) once_load(rsrc_w, woff[j], sw[e], lds_wave, (uint32_t)e * kOnceSlot + (uint32_t)j * 1024u);
    if (lane < 8) *reinterpret_cast<uint4 *>(my_lds + kOnceZeros + lane * 16) = make_uint4(0u, 0u, 0u, 0u);

    // ---- the rows ----
    wait_vmcnt<4 * ST>();
    bool drop = false;
    if (idx) {
        __asm__ volatile("" : "+v"(entry)::"memory");
        p = live ? (int)entry : 0;
    } else if (mask_in) {
        __asm__ volatile("" : "+v"(label)::"memory");
        const bool kept = live && label != 0;
        drop = live && !kept;
        live = kept;
    }
    const bool any = __ballot(live) != 0;
    const SmallUnit u = {waves, wave, mt, nt, group, splits, split, co0, r0, p, live, drop};
    f32x16_t acc;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        __asm__ volatile("" : "+v"(bq[r])::"memory");
        acc[4 * r] = __uint_as_float(bq[r].x); acc[4 * r + 1] = __uint_as_float(bq[r].y);
        acc[4 * r + 2] = __uint_as_float(bq[r].z); acc[4 * r + 3] = __uint_as_float(bq[r].w);
    }
    if (any && busy) {
        const int pp = live ? p : 0;
        const int q = (int)fast_div((uint32_t)pp, g.div_wo), ow = pp - q * g.wo;
        const int img = (int)fast_div((uint32_t)q, g.div_ho), oh = q - img * g.ho;
        const int ih0 = oh * g.sh - g.ph, iw0 = ow * g.sw - g.pw;
        const int pix0 = (img * g.h + ih0) * g.w + iw0; // may lie outside the image

        // the mask bytes under the taps of a kernel row with one (unaligned) 4-byte load each; one that would leave the
        // mask is moved inside it and its bytes moved back (without a mask: three loads of something, not looked at)
        const uint8_t *const from = mask_in ? mask_in : reinterpret_cast<const uint8_t *>(w);
        const int most = mask_in ? g.n * g.h * g.w - 4 : 0; // (positions fit 31 bits)
        uint32_t m[3];
        int moved[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int off = pix0 + k * g.dh * g.w, at = min(max(off, 0), most);
            moved[k] = off - at;
            __asm__ volatile("global_load_dword %0, %1, %2" : "=v"(m[k]) : "v"(at), "s"(from) : "memory");
        }
        // taps inside the image
        uint32_t bits = 0;
        {
            uint32_t cols = 0;
#pragma unroll
            for (int k = 0; k < 3; ++k) cols |= (uint32_t)(iw0 + k) < (uint32_t)g.w ? 1u << k : 0u;
#pragma unroll
            for (int k = 0; k < 3; ++k) bits |= (uint32_t)(ih0 + k * g.dh) < (uint32_t)g.h ? cols << (3 * k) : 0u;
            bits = live ? bits : 0u;
        }
        const u32x4_t rsrc_x = make_rsrc_words(x, (uint32_t)g.n * g.h * g.w * pixel);
        uint32_t xoff[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) xoff[j] = (uint32_t)__shfl(pix0, prow + 8 * j) * pixel + (j & 1 ? piece1 : piece0);

        // ---- weights into registers, pixels into their place ----
        const uint32_t swz = FC_SWZ(l32);
        uint32_t at[4];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) at[kk] = (uint32_t)l32 * 128u + (uint32_t)((2 * kk + half) ^ swz) * 16u;
        Frag<DT> wf[ST][4];
        auto weights = [&](int lo, int hi) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < ST; ++e)
                if (e >= lo && e < hi)
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk) wf[e][kk].load(my_lds + e * kOnceSlot, at[kk]);
        };
        auto pixels = [&](int lo, int hi) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < ST; ++e)
                if (e >= lo && e < hi) {
                    const uint32_t sx = (uint32_t)__builtin_amdgcn_readlane(x_e, e);
#pragma unroll
                    for (int j = 0; j < 4; ++j) once_load(rsrc_x, xoff[j] + sx, 0u, lds_wave, (uint32_t)e * kOnceSlot + (uint32_t)j * 1024u);
                }
        };
        wait_vmcnt<3>(); // the weights have landed (the mask bytes are younger)
        weights(0, 5);
        lds_reads_done();
        weights(5, ST);
        pixels(0, 5);
        lds_reads_done();
        pixels(5, ST);

        // ---- what the mask says about this lane's row under the taps ----
        wait_vmcnt<4 * ST>();
        uint32_t rel = 0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            __asm__ volatile("" : "+v"(m[k])::"memory");
            uint32_t v = moved[k] < 0 ? (moved[k] > -4 ? m[k] << (-8 * moved[k]) : 0u) : (moved[k] < 4 ? m[k] >> (8 * moved[k]) : 0u);
            v = (((v & 0x7f7f7f7fu) + 0x7f7f7f7fu) | v) & 0x80808080u; // nonzero bytes
            rel |= (((v >> 7) & 1u) | ((v >> 14) & 2u) | ((v >> 21) & 4u)) << (3 * k);
        }
        bits &= mask_in ? rel : ~0u;

        // ---- the stages: a stage's pixels are read while the one before is multiplied ----
        Frag<DT> xf[2][4];
#pragma unroll
        for (int e = 0; e <= ST; ++e) {
            if (e < ST) {
                __asm__ volatile("s_waitcnt vmcnt(%0)" : : "n"((ST - 1 - (e < ST ? e : 0)) * 4) : "memory");
                const bool on = bits & (uint32_t)__builtin_amdgcn_readlane(bit_e, e < ST ? e : 0);
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) xf[e & 1][kk].load(my_lds + e * kOnceSlot, on ? at[kk] : kOnceZeros - (uint32_t)e * kOnceSlot);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (e > 1 || (e == 1 && !skip))
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) acc = mfma32<DT>(wf[e > 0 ? e - 1 : 0][kk], xf[(e + 1) & 1][kk], acc);
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
        wait_vmcnt<0>(); // (weights on their way into LDS)
    }
    if (any) small_meet_and_store<DT, TO>(g, u, cut.n_nt, fill, acc, lds, out, partials, tile_counters);
    else if (fill && drop && group == 0) small_clear_tile(g, u, out);
    if (idx && fill) small_clear_rest(g, u, (rows + kSmallRows - 1) / kSmallRows, nts, mask_in, mask_out, out, lds);
}

// ---------------------------------------------------------------------------------------------

static int small_total(const Geom &g) { return g.kh * g.kw * ((g.c_in + 63) / 64); }

// The layers the tiled kernel would run on 64 x 64 tiles: 32-row x 32-channel tiles come to about one
// or two per CU.  Without a list the splits must not depend on the kept count.
bool conv_small_wanted(const Geom &g, int in_dtype, bool room, bool needs_labels)
{
    if (in_dtype != FC_BF16 && in_dtype != FC_F16) return false;
    if (g.flags & (FC_COMPACT_IN | FC_RESIDENT_WEIGHTS)) return false;
    const int taps = g.kh * g.kw, total = small_total(g);
    const int64_t tiles = (int64_t)((g.m + 31) / 32) * ((g.c_out + 31) / 32);
    const int splits = small_splits(1, g.c_out, total, taps, room);
    const int64_t tiles64 = (int64_t)((g.m + 127) / 128) * ((g.c_out + 63) / 64);
    if (taps == 1) {
        // With a list 1x1 kernels are faster elsewhere (576 -> 96 on 16 x 14 x 14 6.3 us, 7.4 here).  Without one, what labels them here is
        // a launch less, or one that ranks all positions in every workgroup, while the tiles are there at once (64 -> 64 on 53 x 33
        // 7.3 -> 4.8 us, 256 -> 1024 on 28 x 28 16.3 -> 6.4, 64 -> 64 on 130 x 130 8.1 -> 6.0; past that, 256 -> 256 on 90 x 90, 2 032 tiles,
        // 10.4 and 13.1), in two rounds where one stage is all they have (64 -> 256 on 90 x 90, 2 032 tiles, 10.6 -> 9.7; 16 ->
        // 224 on 130 x 130, 3 703, 11.3 and 14.8).  Stages count: 256 -> 256 on 64 x 64, 1 024 tiles of four, with 30 % irrelevant 7.6
        // and 7.8, 128 -> 128 on 90 x 90, 1 016 of two, 9.4 -> 6.0.
        // Sums are the same as with a list, so they are cut where the tiled kernel cuts its 64 x 64 tiles, or not at all; past eight
        // stages in one wave there is nothing left to win (768 -> 64 on 28 x 28 8.5 and 8.9; 512 -> 512 9.5 -> 7.4).
        if (!needs_labels || tiles > (total == 1 ? 2048 : (total == 2 ? 1152 : 960))) return false;
        if (total < 2 * kMinSplitStages) return total <= 8;
        return room && tiles64 <= kSmallLayerTiles && tiles * splits <= 1152 && splits == small_splits(g.m, g.c_out, total, taps, room);
    }
    // 3x3: what the tiled kernel would run on 64 x 64 tiles, while a CU gets no more than about four waves
    // (512 -> 512 on 8 x 7 x 7, 1 872 waves, is 14.8 us there and 24.6 us here)
    if (taps == 9 && (tiles64 > kSmallLayerTiles || tiles * splits > kSmallSplitWaves)) return false;
    // Packed reductions without a list: tiles that label their own rows take fewer stages (3x3 where nothing is split here, so that the sums are the same: 16 ->
    // 64 on 28 x 28 7.6 -> 5.2 us, 40 -> 96 7.6 -> 6.1; with splits there is little in it, 72 -> 200 8.3 -> 8.0, 136 -> 136 on 56 x 56 / 2 8.5 -> 8.6).  Other kernels label and gate more taps there: 24 ->
    // 128, 5x5, on 56 x 56 (1 568 waves, 10 stages) 15.6 -> 10.3, 40 -> 96 (1 176, 16) 9.9 -> 11.8; 136 -> 136 (1 960, 54) 25.6 -> 22.1, 80 -> 80 (1 176, 32) 12.3 -> 16.4.
    // Unpacked 64 -> 64, 5x5, on 4 x 48 x 60 (2 880) 21.5 -> 19.6, 192 -> 192 on 56 x 56 (2 352) 27.2 -> 27.9, 128 -> 32 on 4 x 48 x 60 (1 440) 20.3 -> 24.8.
    const bool own_tiles = needs_labels && taps_packed(g, in_dtype, true) && tiles_label_rows(g, in_dtype);
    const int own_stages = reduction_stages(g, in_dtype, true);
    if (taps == 9 && own_tiles && splits == 1) return false;
    if (taps != 9 && (tiles > 1024 || tiles * splits > (own_tiles ? (own_stages <= 16 ? 1200 : 1500) : 2560))) return false;
    return !needs_labels || splits == small_splits(g.m, g.c_out, total, taps, room);
}

// May tiles meet through the workspace (more splits than a workgroup has waves)?
bool conv_small_counts(const Geom &g, bool room) { return small_splits(1, g.c_out, small_total(g), g.kh * g.kw, room) > kSmallWaves; }

// The layers k_conv_small_once serves: 3x3, whole chunks of channels, eight or nine stages a wave whatever is kept, horizontally undilated, mask bytes
// (a row's three taps from one load of four).
static bool small_at_once(const Geom &g, bool room, bool masked)
{
    const int total = small_total(g), splits = small_splits(g.m, g.c_out, total, g.kh * g.kw, room);
    return g.kh == 3 && g.kw == 3 && g.c_in % 64 == 0 && g.dw == 1 && total / splits >= kOnceStages - 1 &&
           (total + splits - 1) / splits <= kOnceStages && splits == small_splits(1, g.c_out, total, 9, room) &&
           (!masked || (!(g.flags & FC_PACKED_MASKS) && (int64_t)g.n * g.h * g.w >= 4));
}

template <int DT, typename TO>
static hipError_t launch_small_t(const Geom &g, bool as_pw, bool room, const void *x, const uint8_t *mask_in, const uint8_t *mask_out,
                                 const void *w, const float *bias, const int32_t *idx, const int32_t *count, void *out,
                                 float *partials, int32_t *tile_counters, hipStream_t s)
{
    const bool once = small_at_once(g, room, mask_in != nullptr);
    const int which = once ? 0 : (as_pw ? 1 : 2);
    auto kern = once ? k_conv_small_once<DT, TO> : (as_pw ? k_conv_small<DT, TO, true> : k_conv_small<DT, TO, false>);
    const uint32_t wave_bytes = once ? kOnceWaveBytes : kSmallWaveBytes;
    const int splits = small_splits(1, g.c_out, small_total(g), g.kh * g.kw, room); // the most any kept count gives
    const int waves = splits < kSmallWaves ? splits : kSmallWaves;
    // (more than 64 KB of dynamic LDS: allowed once per function and device)
    static std::atomic<uint64_t> attr_devices[3] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t dev_bit = 1ull << (dev & 63);
    if (!(attr_devices[which].load(std::memory_order_acquire) & dev_bit)) {
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)(kSmallWaves * wave_bytes));
        if (e != hipSuccess) return e;
        attr_devices[which].fetch_or(dev_bit, std::memory_order_release);
    }
    SmallCut cut;
    cut.n_nt = (g.c_out + kSmallChannels - 1) / kSmallChannels;
    cut.groups = (splits + waves - 1) / waves;
    cut.room = room;
    cut.splits = splits;
    cut.by_splits = make_fastdiv((uint32_t)splits);
    cut.per_mt = make_fastdiv((uint32_t)(cut.n_nt * cut.groups));
    cut.by_groups = make_fastdiv((uint32_t)cut.groups);
    cut.by_kw = make_fastdiv((uint32_t)g.kw);
    cut.by_cch = make_fastdiv((uint32_t)((g.c_in + 63) / 64));
    const int grid = ((g.m + kSmallRows - 1) / kSmallRows) * cut.n_nt * cut.groups;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * waves), waves * wave_bytes, s, g, cut, (const uint16_t *)x, mask_in,
                       mask_out, (const uint16_t *)w, bias, idx, count, (TO *)out, partials, tile_counters);
    return hipGetLastError();
}

hipError_t launch_conv_small(const Geom &g, int in_dtype, int out_dtype, bool as_pw, bool room, const void *x, const uint8_t *mask_in,
                             const uint8_t *mask_out, const void *w, const float *bias, const int32_t *idx,
                             const int32_t *count, void *out, float *partials, int32_t *tile_counters, hipStream_t s)
{
#define FC_SMALL(DT, TO) launch_small_t<DT, TO>(g, as_pw, room, x, mask_in, mask_out, w, bias, idx, count, out, partials, tile_counters, s)
    if (in_dtype == FC_BF16)
        return out_dtype == FC_F32 ? FC_SMALL(FC_BF16, float) : (out_dtype == FC_FP8 ? FC_SMALL(FC_BF16, uint8_t) : FC_SMALL(FC_BF16, uint16_t));
    return out_dtype == FC_F32 ? FC_SMALL(FC_F16, float) : (out_dtype == FC_FP8 ? FC_SMALL(FC_F16, uint8_t) : FC_SMALL(FC_F16, uint16_t));
#undef FC_SMALL
}

} // namespace fc
