// Focused convolution on the matrix cores for layers of a few hundred row blocks (the layers of a
// network at batch 1 to 4; 16-bit storage, more than one tap).
//
// Such a layer is a chain of memory round trips: its matrix work takes a tenth of its time.  This
// kernel is cut for the chain, not for the throughput:
//   - a tile is 32 rows x TN channels, and its reduction is dealt out over the four waves of a
//     workgroup (and, for long reductions, over S workgroups), so no wave multiplies for long;
//   - every wave is a pipeline of its own: it stages its own pixels and weights in its own ring of LDS
//     slots (a slot = 64 channels of one tap for the tile's rows and channels), with no barrier
//     before the sums of the four waves meet;
//   - the tile of a workgroup follows from its number alone, so the weights of its first slots are
//     requested before anything is known about its rows;
//   - with a list, the count and the entries are read together (entries past the count are dropped);
//     without one, a tile is 32 consecutive positions, labelled here: no compaction before the
//     kernel and no zero-fill after it, irrelevant rows come out as zeros;
//   - pixels are gathered as soon as their addresses are known; what the input mask says about
//     them arrives meanwhile and is applied to the operand as it is read from LDS.
// (The tiled kernel took 17 000 cycles for 64 -> 64 at 56 x 56: 1 400 for the count, 4 300 to the rows'
// addresses, 2 000 for the tap bits, 6 100 for nine stages of which 1 150 are matrix instructions.)
#include "fc_dma_util.hpp"
#include <type_traits>
#include <atomic>

namespace fc {

constexpr int kSmallThreads = 256;
constexpr int kSmallRows = 32;
constexpr int kSmallSlots = 3;

template <int TN> constexpr uint32_t small_slot_bytes() { return (uint32_t)(kSmallRows + TN) * 128u; }
template <int TN> constexpr size_t small_lds_bytes() { return (size_t)4 * kSmallSlots * small_slot_bytes<TN>(); }

// How the launch is cut: channel tiles, splits of the reduction, and the division of the workgroup number.
struct SmallCut {
    int32_t n_nt, splits;
    FastDiv per_mt; // by n_nt * splits
    FastDiv by_s;   // by splits
    FastDiv by_cch; // by the 64-channel chunks of a tap
    FastDiv by_kw;
};

template <int DT, typename TO, int TN>
__global__ __launch_bounds__(kSmallThreads, 1) void k_conv_small(Geom g, SmallCut cut, const uint16_t *__restrict__ x,
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
    constexpr int CB = TN / 32;         // 32-channel blocks
    constexpr int XL = kSmallRows / 8;  // wave loads of a slot: 8 rows of 128 bytes each
    constexpr int WL = TN / 8;
    constexpr uint32_t SLOT = small_slot_bytes<TN>();
    extern __shared__ __align__(16) unsigned char lds[];

    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int unit = blockIdx.x, nts = cut.n_nt * cut.splits;
    const int mt = (int)fast_div((uint32_t)unit, cut.per_mt), in_mt = unit - mt * nts;
    const int nt = (int)fast_div((uint32_t)in_mt, cut.by_s), split = in_mt - nt * cut.splits;
    const int co0 = nt * TN, r0 = mt * kSmallRows;
    const int taps = g.kh * g.kw, cch = (g.c_in + 63) >> 6, total = taps * cch;
    // this workgroup's stages [b, e), this wave's [q0, q1)
    const int b = (int)((uint32_t)(split * total) / (uint32_t)cut.splits);
    const int e = (int)((uint32_t)((split + 1) * total) / (uint32_t)cut.splits);
    const int q0 = b + ((wave * (e - b)) >> 2), q1 = b + (((wave + 1) * (e - b)) >> 2), n = q1 - q0;

    const uint32_t lds_wave = __builtin_amdgcn_readfirstlane((uint32_t)reinterpret_cast<uintptr_t>(lds) + (uint32_t)wave * (NS * SLOT));
    const unsigned char *my_lds = lds + (uint32_t)wave * (NS * SLOT);
    const int prow = lane >> 3;
    // (rows of a lane's loads differ by multiples of 8: the swizzle alternates with bit 2 of (row >> 1))
    const int piece0 = (lane & 7) ^ FC_SWZ(prow), piece1 = (lane & 7) ^ FC_SWZ(prow + 8);

    // ---- weights of the first slots ----
    const u32x4_t rsrc_w = make_rsrc_words(w, (uint32_t)g.c_out * taps * g.c_in * 2u);
    auto stage_of = [&](int q, int *tap, int *cc) {
        *tap = (int)fast_div((uint32_t)q, cut.by_cch);
        *cc = q - *tap * cch;
    };
    // (Loops are kept rolled throughout: the kernel runs every instruction once or a few times, so what
    // an unrolled copy costs is the fetching of its code.)
    const int ch0 = piece0 * 8, ch1 = piece1 * 8;
    const uint32_t wrow = (uint32_t)(taps * g.c_in) * 2u;
    const uint32_t woff = (uint32_t)(co0 + prow) * wrow;
    auto load_w = [&](int i) __attribute__((always_inline)) { // slot contents of this wave's stage i
        int tap, cc;
        stage_of(q0 + i, &tap, &cc);
        const uint32_t sw = (uint32_t)(tap * g.c_in + cc * 64) * 2u;
        const int left = i < n ? g.c_in - cc * 64 : 0;
        const uint32_t o0 = ch0 < left ? woff + sw + (uint32_t)ch0 * 2u : kOutOfRange;
        const uint32_t o1 = ch1 < left ? woff + sw + (uint32_t)ch1 * 2u : kOutOfRange;
        uint32_t to = lds_wave + (uint32_t)(i % NS) * SLOT + (uint32_t)kSmallRows * 128u;
        uint32_t row = 0; // rows of weights past the last channel lie past the tensor's end
#pragma unroll 1
        for (int j = 0; j < WL; j += 2) {
            dma_load16(rsrc_w, o0 == kOutOfRange ? o0 : o0 + row, to);
            dma_load16(rsrc_w, o1 == kOutOfRange ? o1 : o1 + row + 8u * wrow, to + 1024u);
            row += 16u * wrow;
            to = __builtin_amdgcn_readfirstlane(to + 2048u);
        }
    };
#pragma unroll 1
    for (int i = 0; i < NS; ++i) load_w(i);

    // ---- the tile's rows: lane l holds row l & 31 ----
    const bool packed = (g.flags & FC_PACKED_MASKS) != 0;
    const bool fill = mask_in && !(g.flags & FC_SKIP_ZERO_FILL);
    int rows = g.m, p = r0 + l32;
    bool live = p < g.m, drop = false;
    if (idx) {
        const int entry = idx[min(p, g.m - 1)];
        rows = *count;
        live = p < rows;
        p = live ? entry : 0;
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
        auto load_x = [&](int i) __attribute__((always_inline)) {
            int tap, cc;
            stage_of(q0 + i, &tap, &cc);
            const int kh = (int)fast_div((uint32_t)tap, cut.by_kw), kw = tap - kh * g.kw;
            const uint32_t sx = __builtin_amdgcn_readfirstlane((uint32_t)((kh * g.dh * g.w + kw * g.dw) * g.c_in + cc * 64) * 2u);
            const uint32_t to = lds_wave + (uint32_t)(i % NS) * SLOT;
            const int left = i < n ? g.c_in - cc * 64 : 0;
            const uint32_t sel0 = ch0 < left ? 1u << (tap & 31) : 0u, sel1 = ch1 < left ? 1u << (tap & 31) : 0u;
#pragma unroll
            for (int j = 0; j < XL; ++j)
                dma_load16(rsrc_x, (xin[j] & (j & 1 ? sel1 : sel0)) ? xoff[j] + sx : kOutOfRange,
                           __builtin_amdgcn_readfirstlane(to + (uint32_t)j * 1024u));
        };
#pragma unroll 1
        for (int i = 0; i < NS; ++i) load_x(i);

        // what the mask says about this lane's row under the wave's taps
        uint32_t bits = inside;
        if (mask_in) {
            int t0, t1, cc;
            stage_of(q0, &t0, &cc);
            stage_of(n > 0 ? q1 - 1 : q0, &t1, &cc);
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

        f32x16_t acc[CB];
#pragma unroll
        for (int c = 0; c < CB; ++c)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[c][i] = 0.f;
        const uint32_t frag = (uint32_t)l32 * 128u, swz = FC_SWZ(l32);
        wait_vmcnt<0>(); // the first NS slots
#pragma unroll 1
        for (int i = 0; i < n; ++i) {
            wait_vmcnt<(XL + WL) * (NS - 1)>(); // slot i (later ones are behind it)
            int tap, cc;
            stage_of(q0 + i, &tap, &cc);
            const unsigned char *xs = my_lds + (uint32_t)(i % NS) * SLOT + frag, *ws = xs + kSmallRows * 128;
            Frag<DT> xf[4], wf[4][CB];
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                const uint32_t o = (uint32_t)((2 * kk + half) ^ swz) * 16u;
                xf[kk].load(xs, o);
#pragma unroll
                for (int c = 0; c < CB; ++c) wf[kk][c].load(ws + c * 4096, o);
            }
            __builtin_amdgcn_sched_barrier(0); // all operands of the slot in flight before the first multiply
            const bool on = (bits >> (tap & 31)) & 1u;
            const int ks = min(4, (g.c_in - cc * 64 + 15) >> 4); // 16-channel steps that exist
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                if (kk >= ks) break;
                xf[kk].v.x = on ? xf[kk].v.x : 0u;
                xf[kk].v.y = on ? xf[kk].v.y : 0u;
                xf[kk].v.z = on ? xf[kk].v.z : 0u;
                xf[kk].v.w = on ? xf[kk].v.w : 0u;
#pragma unroll
                for (int c = 0; c < CB; ++c) acc[c] = mfma32<DT>(wf[kk][c], xf[kk], acc[c]);
            }
            // the slot's next contents (past the end: loads that are switched off, so that the counts of the
            // waits hold)
            __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            load_w(i + NS);
            load_x(i + NS);
        }
        wait_vmcnt<0>();

        // ---- the waves' sums meet: quad (c, q) of a lane = channels 32 c + 8 q + 4 half .. + 3 of its row ----
        __syncthreads();
        float4 *part = reinterpret_cast<float4 *>(lds);
#pragma unroll
        for (int c = 0; c < CB; ++c)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                part[((wave * CB + c) * 4 + q) * 64 + lane] =
                    make_float4(acc[c][4 * q], acc[c][4 * q + 1], acc[c][4 * q + 2], acc[c][4 * q + 3]);
        __syncthreads();
        float4 v[CB]; // wave q finishes quad q of every block
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            v[c] = part[(c * 4 + wave) * 64 + lane];
#pragma unroll
            for (int k = 1; k < 4; ++k) {
                const float4 t = part[((k * CB + c) * 4 + wave) * 64 + lane];
                v[c].x += t.x; v[c].y += t.y; v[c].z += t.z; v[c].w += t.w;
            }
        }
        bool mine = true;
        if (cut.splits > 1) {
            // Park the sums (device-scope accesses, as in the tiled kernel), count in; the workgroup that
            // arrives last adds the S partial tiles in split order.
            const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(
                partials, 0, (uint32_t)((size_t)kSplitGrid * kSplitTileFloats * sizeof(float)), 0x00020000);
            constexpr uint32_t TILE = (uint32_t)kSmallRows * TN * 4u;
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                u32x4_t t;
                t.x = __float_as_uint(v[c].x); t.y = __float_as_uint(v[c].y);
                t.z = __float_as_uint(v[c].z); t.w = __float_as_uint(v[c].w);
                __builtin_amdgcn_raw_buffer_store_b128(t, rp, (uint32_t)unit * TILE + (uint32_t)(c * 256 + tid) * 16u, 0, kDeviceScope);
            }
            wait_vmcnt<0>();
            __syncthreads();
            int *arrived = reinterpret_cast<int *>(lds + 4 * CB * 4 * 64 * 16);
            const int tile = mt * cut.n_nt + nt;
            if (tid == 0)
                *arrived = __hip_atomic_fetch_add(&tile_counters[tile], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            mine = *arrived == cut.splits - 1;
            if (mine) {
                if (tid == 0) // leave the counters as they were found
                    __hip_atomic_store(&tile_counters[tile], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const uint32_t first = (uint32_t)(unit - split) * TILE;
#pragma unroll
                for (int c = 0; c < CB; ++c) v[c] = make_float4(0.f, 0.f, 0.f, 0.f);
                constexpr int U = 4; // partial tiles in flight
                for (int s0 = 0; s0 < cut.splits; s0 += U) {
                    u32x4_t t[U][CB];
#pragma unroll
                    for (int u = 0; u < U; ++u)
#pragma unroll
                        for (int c = 0; c < CB; ++c)
                            t[u][c] = __builtin_amdgcn_raw_buffer_load_b128(
                                rp, s0 + u < cut.splits ? first + (uint32_t)(s0 + u) * TILE + (uint32_t)(c * 256 + tid) * 16u : kOutOfRange,
                                0, kDeviceScope);
#pragma unroll
                    for (int u = 0; u < U; ++u)
#pragma unroll
                        for (int c = 0; c < CB; ++c) {
                            v[c].x += __uint_as_float(t[u][c].x); v[c].y += __uint_as_float(t[u][c].y);
                            v[c].z += __uint_as_float(t[u][c].z); v[c].w += __uint_as_float(t[u][c].w);
                        }
                }
            }
        }
        if (mine && (live || (drop && fill))) {
            const int64_t orow = (g.flags & FC_COMPACT_OUT) ? (int64_t)r0 + l32 : (int64_t)(drop ? r0 + l32 : p);
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                const int co = co0 + c * 32 + wave * 8 + half * 4;
                if (co >= g.c_out) continue;
                float4 t = v[c];
                if (bias) {
                    const float4 bq = *reinterpret_cast<const float4 *>(bias + co);
                    t.x += bq.x; t.y += bq.y; t.z += bq.z; t.w += bq.w;
                }
                if (drop) t = make_float4(0.f, 0.f, 0.f, 0.f);
                TO *o = out + orow * g.c_out + co;
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
            }
        }
    } else {
        wait_vmcnt<0>(); // (weights on their way into LDS)
        if (fill && drop && split == 0) { // 32 irrelevant positions: wave v clears every fourth 16-byte piece
            const int pieces = min(TN, g.c_out - co0) * (int)sizeof(TO) / 16;
            const u32x4_t zero = {0u, 0u, 0u, 0u};
            for (int i = wave * 2 + half; i < pieces; i += 8)
                *reinterpret_cast<u32x4_t *>(out + (int64_t)(r0 + l32) * g.c_out + co0 + i * (16 / (int)sizeof(TO))) = zero;
        }
    }

    // with a list: the irrelevant rows, by the workgroups whose tile does not exist when there are enough
    if (idx && fill) {
        const int grid = gridDim.x, idle = grid - tiles * nts;
        const bool idle_only = idle * 16 >= grid;
        if (!idle_only || mt >= tiles) {
            if (any) __syncthreads(); // LDS is free again
            clear_irrelevant(g, mask_in, mask_out, out, g.c_out * (int)sizeof(TO) / 16,
                             (idle_only ? unit - tiles * nts : unit) * 4 + wave, (idle_only ? idle : grid) * 4,
                             reinterpret_cast<int32_t *>(lds) + wave * 64);
        }
    }
}

// ---------------------------------------------------------------------------------------------

static int small_total(const Geom &g) { return g.kh * g.kw * ((g.c_in + 63) / 64); }

// Layers whose 32-row x 64-channel tiles come to about one workgroup per CU (its slots fill most of a CU's
// LDS).  Measured against the tiled kernel on half-kept layers, call without a list / with a list / no mask:
// 64 -> 64 at 56 x 56 9.0 / 7.5 / 7.0 -> 6.0 / 5.7 / 5.3 us, 512 -> 512 at 7 x 7 14.3 / 11.6 / 11.3 -> 8.7 / 8.3 / 8.0 us;
// 128 -> 128 on 8 x 28 x 28 (392 tiles) 15.8 / 11.9 / 11.9 -> 18.3 / 11.2 / 15.2 us, so the line lies below that.
bool conv_small_wanted(const Geom &g, int in_dtype)
{
    if (in_dtype != FC_BF16 && in_dtype != FC_F16) return false;
    if (g.kh * g.kw == 1 || (g.flags & (FC_COMPACT_IN | FC_RESIDENT_WEIGHTS))) return false;
    return (int64_t)((g.m + 31) / 32) * ((g.c_out + 63) / 64) <= 320;
}

// Splits of the reduction over workgroups: only where it is so long that the weights of a tile, at
// the 64 bytes a cycle a CU can take in, cost more than the exchange of partial sums (about 4 000 cycles).
int conv_small_splits(const Geom &g, bool room)
{
    const int total = small_total(g);
    const int tiles = ((g.m + 31) / 32) * ((g.c_out + 63) / 64);
    if (!room || total < 36) return 1;
    int s = total / 18;
    while (s > 1 && tiles * s > 256) --s; // (one workgroup per CU)
    return s > 8 ? 8 : s;
}

template <int DT, typename TO, int TN>
static hipError_t launch_small_t(const Geom &g, int splits, const void *x, const uint8_t *mask_in, const uint8_t *mask_out,
                                 const void *w, const float *bias, const int32_t *idx, const int32_t *count, void *out,
                                 float *partials, int32_t *tile_counters, hipStream_t s)
{
    auto kern = k_conv_small<DT, TO, TN>;
    constexpr size_t bytes = small_lds_bytes<TN>();
    // (more than 64 KB of dynamic LDS: allowed once per function and device)
    static std::atomic<uint64_t> attr_devices{0};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t dev_bit = 1ull << (dev & 63);
    if (!(attr_devices.load(std::memory_order_acquire) & dev_bit)) {
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        if (e != hipSuccess) return e;
        attr_devices.fetch_or(dev_bit, std::memory_order_release);
    }
    SmallCut cut;
    cut.n_nt = (g.c_out + TN - 1) / TN;
    cut.splits = splits;
    cut.per_mt = make_fastdiv((uint32_t)(cut.n_nt * splits));
    cut.by_s = make_fastdiv((uint32_t)splits);
    cut.by_kw = make_fastdiv((uint32_t)g.kw);
    cut.by_cch = make_fastdiv((uint32_t)((g.c_in + 63) / 64));
    const int grid = ((g.m + kSmallRows - 1) / kSmallRows) * cut.n_nt * splits;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kSmallThreads), bytes, s, g, cut, (const uint16_t *)x, mask_in, mask_out,
                       (const uint16_t *)w, bias, idx, count, (TO *)out, partials, tile_counters);
    return hipGetLastError();
}

template <int DT, typename TO>
static hipError_t launch_small_o(const Geom &g, int splits, const void *x, const uint8_t *mask_in, const uint8_t *mask_out,
                                 const void *w, const float *bias, const int32_t *idx, const int32_t *count, void *out,
                                 float *partials, int32_t *tile_counters, hipStream_t s)
{
    // 32 channels per tile while that is no more than a workgroup per CU: half the work each (64 -> 64 at
    // 56 x 56 7.2 -> 6.0 us; 256 -> 256 on 8 x 14 x 14, 392 such tiles, 11.2 -> 16.6 us)
    if (((g.m + 31) / 32) * ((g.c_out + 31) / 32) * splits > 256)
        return launch_small_t<DT, TO, 64>(g, splits, x, mask_in, mask_out, w, bias, idx, count, out, partials, tile_counters, s);
    return launch_small_t<DT, TO, 32>(g, splits, x, mask_in, mask_out, w, bias, idx, count, out, partials, tile_counters, s);
}

hipError_t launch_conv_small(const Geom &g, int in_dtype, int out_dtype, int splits, const void *x, const uint8_t *mask_in,
                             const uint8_t *mask_out, const void *w, const float *bias, const int32_t *idx,
                             const int32_t *count, void *out, float *partials, int32_t *tile_counters, hipStream_t s)
{
#define FC_SMALL(DT, TO) launch_small_o<DT, TO>(g, splits, x, mask_in, mask_out, w, bias, idx, count, out, partials, tile_counters, s)
    if (in_dtype == FC_BF16)
        return out_dtype == FC_F32 ? FC_SMALL(FC_BF16, float) : (out_dtype == FC_FP8 ? FC_SMALL(FC_BF16, uint8_t) : FC_SMALL(FC_BF16, uint16_t));
    return out_dtype == FC_F32 ? FC_SMALL(FC_F16, float) : (out_dtype == FC_FP8 ? FC_SMALL(FC_F16, uint8_t) : FC_SMALL(FC_F16, uint16_t));
#undef FC_SMALL
}

} // namespace fc
