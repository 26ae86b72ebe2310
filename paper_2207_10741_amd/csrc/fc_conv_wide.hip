// Focused 3x3 convolution on the gfx950 matrix cores, tiles of up to 256 x 256 or 384 x 128 per CU (Sec. III-A: a
// GEMM over the kept patches only, with the dense layer's weights).
//
// Same GEMM view and data path as the tiled kernel next door (rows = kept output positions, reduction = (kernel row,
// 128-byte chunk of channels, horizontal tap), gathers straight from global memory into swizzled LDS rows, the pixel
// line shared by the three horizontal taps, 32x32 matrix instructions, sums that start from the bias), for layers
// with enough rows to give every CU several tiles.  The tiled kernel's 64 x 64 wave tiles read 1 KB of fragments a matrix
// instruction and write a weight slab for every 128 rows; its matrix pipes are busy 62 % of the cycles, at a clock that the
// power of all this holds at 1.73 GHz (256 -> 256 on 8 x 270 x 480 without a mask).  Here one workgroup of eight waves per CU
// owns 256 x 256 outputs (8-bit: 192 x 256) or 384 x 128, a wave 128 x 64: 0.75 KB a matrix instruction, a slab for 256
// rows, a third of the barriers.  Pipes busy 74 %, 1.66 GHz; the same layer 1 088 -> 946 us (1.12 -> 1.28 PFLOP/s).  (Four waves of 128 x
// 128, one a SIMD: 0.5 KB an instruction, but every wait is exposed: busy 60 %, 1.9 .. 2.0 GHz, 964 .. 1 007 us.)
//
// Nothing stands in the way of the products: fragments are read a k-step ahead, across the stage boundary as well (the barrier
// stands inside the last k-step of a stage, whose remaining products cover the first reads of the next one), every read and
// load goes out between two products (in bursts between the k-steps: 1 126 us with four waves, 964 so), a stage's slab is
// sent for a stage ahead, a line two.  A stage of one or two granules lasts less than a round trip, so 256-channel tiles of at most
// two, whose lines are short, keep a third slab in the room behind them and send for slabs two stages ahead (512 -> 512 on 128 x 16 x 16, chained,
// 0.1 / 0.2 kept 49 / 57 -> 43 / 46 us; 128-channel tiles, whose slabs are half as large, +1 %).
//
// Tiles are made of granules of WM * 32 rows; XCD j takes the j-th eighth of the granules and deals them to its workgroups side by
// side, every workgroup the same number but for one, in as few rounds as tiles of PBX granules allow and all rounds alike: 4.7 granules
// a workgroup are two tiles of two or three, not one of four and one of one, whose stages would last no less than a round
// trip (256 -> 256 on 16 x 60 x 80 without a mask 92 -> 88 .. 91 us).  A tile whose pixel line would not fit (a fragmented mask)
// gathers its rows tap by tap instead, into the same buffers, a buffer of rows a stage; the order of the sums is the same.  (With
// fewer granules per tile instead: 512 -> 512 on 128 x 16 x 16, 0.3 kept at random, 110 us, so 64; 256 -> 256 on 128 x 32 x 32 87, so 51.)
//
// Irrelevant rows are cleared inside the loop: every tile comes with a range of positions, whose labels it reads in its
// set-up, and a stage's stores go out at its end.  Loads and stores count in one counter and come back in order, so the waits
// for loads let the stores that went out after them be (as if they were not there, a store had one stage to complete).  Workgroups that
// the longest quota leaves without a tile only clear.  Zero-filled layers that keep little, before -> so: 128 -> 128 on
// 128 x 64 x 64, 0.1 / 0.2 kept 44.5 / 61 -> 33 / 52 us, 256 -> 256 on 128 x 32 x 32 36 / 48 -> 32 / 42.
#include "fc_dma_util.hpp"
#include <atomic>
#include <type_traits>

namespace fc {

constexpr int kWideWaves = 8, kWideThreads = kWideWaves * 64;
constexpr int kWideWords = 3; // positions a tile clears: up to 64 * 3 per wave

// SLS > 0: tiles of at most two granules have three slabs instead of two.  The third lies behind their lines, which are at most
// SLS slots long (or three buffers of rows).
template <int WM, int TN, int SL, int SLS>
constexpr uint32_t wide_x_bytes()
{
    constexpr uint32_t two = 2u * SL * 128u, line3 = 2u * SLS * 128u + TN * 128u, rows3 = 3u * 2u * WM * 32u * 128u + TN * 128u;
    constexpr uint32_t three = line3 > rows3 ? line3 : rows3;
    return SLS > 0 && three > two ? three : two;
}

template <int WM, int TN, int PBX, int SL, int SLS>
constexpr size_t wide_lds_bytes()
{
    return wide_x_bytes<WM, TN, SL, SLS>() + (size_t)2 * TN * 128 + (size_t)(2 * WM * PBX * 32 + 3 * SL + 32) * sizeof(int32_t) + (size_t)kWideWords * kWideWaves * 8;
}

// f(integral_constant 0) .. f(integral_constant N - 1)
template <int N, int I = 0, typename F> __device__ __forceinline__ void steps(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        steps<N, I + 1>(f);
    }
}

struct WideArgs {
    int32_t n_nt;   // channel tiles
    FastDiv cpr;    // 16-byte pieces per output row
};

// DT: storage type; TO: float or the 16-bit / 8-bit carrier of the output; WM x WN waves (eight); TN = WN * 64 output channels; PBX: most
// 32-row blocks of a wave; SL: slots of a pixel line.
template <int DT, typename TO, int WM, int PBX, int SL, int SLS>
__global__ __launch_bounds__(kWideThreads, 2)
void k_conv_wide(Geom g, WideArgs wa, const unsigned char *__restrict__ x, const uint8_t *__restrict__ mask_in,
                 const uint8_t *__restrict__ mask_out, const unsigned char *__restrict__ w, const float *__restrict__ bias,
                 const int32_t *__restrict__ idx, const int32_t *__restrict__ count, TO *__restrict__ out)
{
    constexpr int NT = kWideThreads, WN = kWideWaves / WM, CB = 2, TN = WN * CB * 32, TM = WM * PBX * 32, GR = WM * 32; // GR: rows of a granule
    constexpr int ES = DT == FC_FP8 ? 1 : 2, TK = kStageBytes / ES;
    constexpr int ODT = DT == FC_FP8 ? FC_BF16 : DT;
    constexpr uint32_t KSTEP = kStepBytes<DT>;
    constexpr int KK = kStageBytes / (int)KSTEP;
    constexpr int RPL = NT / 8;                         // LDS rows the eight waves' loads cover side by side
    constexpr int WL = TN / RPL;                       // wave loads per wave: a slab
    constexpr int SIT = (SL + NT - 1) / NT;
    constexpr uint32_t WB = (uint32_t)TN * 128u, HALF = KSTEP / 32u;
    constexpr uint32_t W0 = wide_x_bytes<WM, TN, SL, SLS>(); // slabs 0 and 1 lie from here on, slab 2 right below
    static_assert(SL % RPL == 0 && SLS % RPL == 0 && SL >= TM && (SLS == 0 || SLS >= 2 * GR) && TM <= NT, "whole wave loads; rows fit where lines do; one row a thread");

    extern __shared__ __align__(16) unsigned char smem_raw[];
    const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>(smem_raw);
    int32_t *row_p = reinterpret_cast<int32_t *>(smem_raw + W0 + 2 * WB);
    int32_t *row_cs = row_p + TM;
    int32_t *slot_pix = row_cs + TM;
    int32_t *slot_hw = slot_pix + SL;
    uint32_t *slot_bits = reinterpret_cast<uint32_t *>(slot_hw + SL);
    int32_t *scan_part = reinterpret_cast<int32_t *>(slot_bits + SL); // [8] wave totals
    uint64_t *drop = reinterpret_cast<uint64_t *>(scan_part + 32);     // [kWideWords][8] irrelevant ones of the positions to clear

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // (what follows from the thread number alone is computed per tile: kept for the whole kernel it takes the registers
    // of the loop)
    auto thread_number = [&]() __attribute__((always_inline)) {
        int v = threadIdx.x;
        __asm__ volatile("" : "+v"(v));
        return v;
    };
    const int wave_m = wave % WM, wave_n = wave / WM;
    const bool packed_masks = (g.flags & FC_PACKED_MASKS) != 0;
    int rows = g.m;
    if (idx) rows = *count;
    rows = __builtin_amdgcn_readfirstlane(rows);

    const int cchunks = g.c_in / TK, groups = 3 * cchunks;
    const u32x4_t rsrc_w = make_rsrc_words(w, (uint32_t)g.c_out * 9u * (uint32_t)g.c_in * (uint32_t)ES);
    // (a slot's offset is that of its first kernel row, which may lie above the image: the line is gathered through a
    // descriptor that starts pad_h rows + pad_w pixels before the tensor; nothing in front of the tensor is read)
    const uint32_t xbias = (uint32_t)(g.ph * g.w + g.pw) * (uint32_t)g.c_in * (uint32_t)ES;
    const u32x4_t rsrc_x = make_rsrc_words(x - xbias, (uint32_t)g.n * g.h * g.w * g.c_in * (uint32_t)ES + xbias);
    const uint32_t lds_wave = lds0 + (uint32_t)wave * 1024u;

    // ---- granules: (channel tile, row granule) pairs, channel tile first ----
    const int nb = (rows + GR - 1) / GR, total = nb * wa.n_nt;
    const int xcd = (int)blockIdx.x & 7, slot_x = (int)blockIdx.x >> 3, per_xcd = (int)gridDim.x >> 3;
    const int x0 = (int)(((int64_t)total * xcd) >> 3), x1 = (int)(((int64_t)total * (xcd + 1)) >> 3);
    // (with rows to clear no more workgroups take tiles than the longest quota needs: 410 granules are two each for 205 of 256, and
    // the others only clear)
    const bool zero_fill = mask_in && !(g.flags & FC_SKIP_ZERO_FILL);
    const int n_x = x1 - x0, qm = (n_x + per_xcd - 1) / per_xcd;
    const int takers = zero_fill ? (qm > 0 ? (n_x + qm - 1) / qm : 0) : per_xcd, clearers = per_xcd - takers;
    // a workgroup's quota is q granules or q + 1 (extra: how many of the workgroups before it have one more), cut into rounds
    const int q = takers > 0 ? n_x / takers : 0, rem = n_x - q * takers, rounds = (qm + PBX - 1) / PBX;
    const int extra = takers > 0 ? (slot_x * rem) / takers : 0, mine = takers > 0 ? q + ((slot_x + 1) * rem) / takers - extra : 0;

    // ---- zero-fill: an XCD clears the j-th eighth of the positions (all channels).  A workgroup without tiles clears what two with
    // tiles do; a granule comes with zq positions, or where those are too many (masks that keep little) its share is cleared
    // at the end ----
    const int cpr = g.c_out * (int)sizeof(TO) / 16;
    int zx0 = 0, zx1 = 0, zt0 = 0, zq = 0;
    bool clear_in_loop = false;
    if (zero_fill) {
        zx0 = (int)(((int64_t)g.m * xcd) >> 3);
        zx1 = (int)(((int64_t)g.m * (xcd + 1)) >> 3);
        zt0 = n_x > 0 ? zx0 + (zx1 - zx0) / (2 * clearers + takers) * (2 * clearers) : zx1;
        zq = n_x > 0 ? (zx1 - zt0 + n_x - 1) / n_x : 0;
        clear_in_loop = n_x > 0 && (int64_t)zq * ((qm + rounds - 1) / max(rounds, 1)) <= kWideWords * NT;
    }
    if (zero_fill && slot_x >= takers)
        clear_irrelevant_runs(g, mask_in, mask_out, out, cpr, wa.cpr, zx0, zt0, (slot_x - takers) * kWideWaves + wave, clearers * kWideWaves);

    for (int round = slot_x < takers ? 0 : rounds; round < rounds; ++round) {
        const int qa = (q * round) / rounds, qb = ((q + 1) * round) / rounds; // granules of the rounds before, per workgroup of either kind
        const int ca = (q * (round + 1)) / rounds - qa, cb = ((q + 1) * (round + 1)) / rounds - qb;
        int g0 = x0 + (takers - rem) * qa + rem * qb + (slot_x - extra) * ca + extra * cb;
        const int g1 = g0 + (mine > q ? cb : ca);
        while (g0 < g1) {
            const int nt = g0 / nb, rg = g0 - nt * nb;
            const int k = min(min(g1 - g0, nb - rg), PBX);
            const int co0 = nt * TN, m0 = rg * GR;
            const int tid = thread_number(), lane = tid & 63, slot8 = lane & 7;
            // fragment addressing as in the tiled kernel
            const uint32_t frag_row = (uint32_t)(lane & 31) * 128u;
            const uint32_t frag_t16 = (uint32_t)(((lane >> 5) * HALF) ^ FC_SWZ(lane & 31)) * 16u;

            // weight cursor and slabs: the first two are sent for before the set-up (nobody reads them any more)
            const uint32_t wrow = 9u * (uint32_t)g.c_in * (uint32_t)ES; // bytes of a channel's weights
            const int wr0 = wave * 8 + (lane >> 3);
            const uint32_t woff = (uint32_t)(co0 + wr0) * wrow + (uint32_t)(slot8 ^ FC_SWZ(wr0)) * 16u;
            int wkh = 0, wcc = 0, wkw = 0, wleft = 3 * groups;
            uint32_t ld_sw = 0;
            // (slabs past the last one: the first one again, which nobody reads)
            auto next_w = [&]() __attribute__((always_inline)) {
                ld_sw = wleft > 0 ? (uint32_t)((wkh * 3 + wkw) * g.c_in + wcc * TK) * (uint32_t)ES : 0u;
                --wleft;
                const int w3 = (wkw == 2);
                wkw = w3 ? 0 : wkw + 1;
                const int wc = w3 & (wcc + 1 == cchunks);
                wcc = w3 ? (wc ? 0 : wcc + 1) : wcc;
                wkh += wc;
            };
            auto issue_w = [&](int j, uint32_t buf) __attribute__((always_inline)) {
                dma_load16_any(rsrc_w, woff, ld_sw + (uint32_t)j * RPL * wrow, lds_wave + W0 + (buf < 2 ? buf * WB : 0u - WB) + (uint32_t)j * (RPL * 128u));
            };
            __syncthreads(); // the previous tile is done with LDS
#pragma unroll
            for (int d = 0; d < 2; ++d) {
                next_w();
#pragma unroll
                for (int j = 0; j < WL; ++j) issue_w(j, (uint32_t)d);
            }

            // ---- set-up: rows -> slots of the pixel line -> tap bits; the labels of the positions to clear ----
            // (one row a thread)
            const bool live = tid < k * GR && m0 + tid < rows;
            const int m = m0 + tid;
            const int sp = live ? (idx ? idx[m] : m) : -1;
            const int prev = (live && tid > 0) ? (idx ? idx[m - 1] : m - 1) : -2;
            const int next = (live && tid + 1 < k * GR && m + 1 < rows) ? (idx ? idx[m + 1] : m + 1) : -2;
            const int sq = (int)fast_div((uint32_t)max(sp, 0), g.div_wo);
            const int sow = max(sp, 0) - sq * g.wo;
            const int sb = (int)fast_div((uint32_t)sq, g.div_ho);
            const int sih = (sq - sb * g.ho) * g.sh - g.ph;
            const bool ladj = live && prev == sp - 1 && sow > 0;
            const bool radj = live && next == sp + 1 && sow < g.wo - 1;
            // (the pixel between two kept positions with one dropped between them has one slot, the right of the one and the left of the
            // other: 0.9 kept at random, 128 -> 128 on 128 x 64 x 64 155 -> 146 us, 256 -> 256 on 128 x 32 x 32 126 -> 117)
            const int lead = live && !ladj && !(prev == sp - 2 && sow > 1), cnt = tid < k * GR ? 1 + lead + (live && !radj) : 0;
            const int incl = wave_inclusive_scan(cnt);
            if (lane == 63) scan_part[wave] = incl;
            if (tid < TM) row_p[tid] = live && (g.flags & FC_COMPACT_OUT) ? m : sp; // where the row goes
            const int z0 = clear_in_loop ? min(zt0 + (g0 - x0) * zq, zx1) : 0;
            const int zl = clear_in_loop ? min(k * zq, zx1 - z0) : 0; // positions this tile clears
            {
                bool kept[kWideWords];
#pragma unroll
                for (int i = 0; i < kWideWords; ++i) {
                    const int p = z0 + i * NT + tid;
                    kept[i] = true;
                    if (i * NT + tid < zl) kept[i] = position_kept(g, mask_in, mask_out, p);
                }
#pragma unroll
                for (int i = 0; i < kWideWords; ++i) {
                    const uint64_t d = __ballot(!kept[i]);
                    if (lane == 0) drop[i * kWideWaves + wave] = d;
                }
            }
            __syncthreads();
            int ns = 1, before = 0; // slots of the line (a row past the end reads the slot after its own as well)
#pragma unroll
            for (int v = 0; v < kWideWaves; ++v) {
                const int t = scan_part[v];
                before += v < wave ? t : 0;
                ns += t;
            }
            ns = __builtin_amdgcn_readfirstlane(ns);
            // A line that does not fit (a fragmented mask): the rows are gathered tap by tap, into the same buffers.
            const bool by_tap = ns > (SLS > 0 && k <= 2 ? SLS : SL);
            const int iwc = sow - g.pw + 1;
            const int pixc = (sb * g.h + sih) * g.w + iwc;
            if (by_tap) {
                // (the nine bytes of a row are in flight together)
                uint32_t bits = 0;
                bool in[9], on[9];
#pragma unroll
                for (int t = 0; t < 9; ++t) {
                    const int ih = sih + t / 3 * g.dh, iw = iwc - 1 + t % 3;
                    in[t] = live && (uint32_t)ih < (uint32_t)g.h && (uint32_t)iw < (uint32_t)g.w;
                    on[t] = true;
                }
                if (mask_in) {
#pragma unroll
                    for (int t = 0; t < 9; ++t) on[t] = mask_at(mask_in, in[t] ? pixc - 1 + t / 3 * g.dh * g.w + t % 3 : 0, packed_masks);
                }
#pragma unroll
                for (int t = 0; t < 9; ++t) bits |= (uint32_t)(in[t] && on[t]) << t;
                if (tid < TM) {
                    slot_pix[tid] = live ? pixc - 1 : 0;
                    slot_bits[tid] = bits;
                }
            } else {
                const int cs = before + incl - cnt + lead;
                const int ih16 = (int)((uint32_t)sih & 0xffffu);
                if (tid < k * GR) {
                    row_cs[tid] = cs;
                    if (live) {
                        slot_pix[cs] = pixc;
                        slot_hw[cs] = ih16 | (int)((uint32_t)iwc << 16);
                        if (!ladj) {
                            slot_pix[cs - 1] = pixc - 1;
                            slot_hw[cs - 1] = ih16 | (int)((uint32_t)(iwc - 1) << 16);
                        }
                        if (!radj) {
                            slot_pix[cs + 1] = pixc + 1;
                            slot_hw[cs + 1] = ih16 | (int)((uint32_t)(iwc + 1) << 16);
                        }
                    } else {
                        slot_pix[cs] = 0;
                        slot_hw[cs] = (int)((uint32_t)(-20000) << 16); // never inside an image
                    }
                }
                __syncthreads();
#pragma unroll
                for (int i = 0; i < SIT; ++i) {
                    const int sl = tid + i * NT;
                    const bool used = sl < ns - 1;
                    const int hw = used ? slot_hw[sl] : 0, pix = used ? slot_pix[sl] : 0;
                    const int ih0 = (int)(int16_t)(hw & 0xffff), iw = hw >> 16;
                    bool in[3];
                    bool on[3];
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        const int ih = ih0 + q * g.dh;
                        in[q] = used && ih >= 0 && ih < g.h && iw >= 0 && iw < g.w;
                        on[q] = in[q];
                    }
                    if (mask_in) {
                        uint32_t rel[3];
#pragma unroll
                        for (int q = 0; q < 3; ++q) rel[q] = mask_at(mask_in, in[q] ? pix + q * g.dh * g.w : 0, packed_masks);
                        loaded_together(rel);
#pragma unroll
                        for (int q = 0; q < 3; ++q) on[q] = on[q] && rel[q];
                    }
                    if (sl < SL) {
                        slot_bits[sl] = (uint32_t)on[0] | (uint32_t)on[1] << 1 | (uint32_t)on[2] << 2;
                        if (!used) slot_pix[sl] = 0;
                    }
                }
            }
            __syncthreads();
            const int nxl = (ns + RPL - 1) / RPL; // loads of a line

            // PB: 32-row blocks of a wave (granules of the tile); TAP: gathered tap by tap
            auto run = [&](auto pb_c, auto tap_c) __attribute__((always_inline)) {
                constexpr int PB = decltype(pb_c)::value;
                constexpr bool TAP = decltype(tap_c)::value;
                constexpr int R = SLS > 0 && PB <= 2 ? 3 : 2;                          // slabs, and buffers of rows
                constexpr int XL = TAP ? PB * GR / RPL : (R == 3 ? SLS : SL) / RPL;    // wave loads per wave: rows, a line
                constexpr uint32_t XB = (TAP ? PB * GR : (R == 3 ? SLS : SL)) * 128u;  // a buffer of theirs
                constexpr int NG = TAP ? 9 : 3, PW = TAP ? 3 : 10;                     // gates per slot (row) this lane gathers; of them a word holds
                static_assert((TAP ? R : 2) * XB + (R - 2) * WB <= W0, "buffers of rows and the third slab");
                // (a short line is sent for whole, whatever it holds: the waits then know its loads)
                constexpr bool WHOLE = TAP || XL <= 3;
                uint32_t hxoff[XL];
                uint32_t hxbits[2] = {0, 0};
                static_assert(XL <= 2 * PW, "two words");
#pragma unroll
                for (int j = 0; j < XL; ++j) {
                    const int sl = j * RPL + wave * 8 + (lane >> 3);
                    hxoff[j] = (uint32_t)slot_pix[sl] * (uint32_t)(g.c_in * ES) + (uint32_t)(slot8 ^ FC_SWZ(sl)) * 16u + xbias;
                    hxbits[j / PW] |= slot_bits[sl] << (NG * (j % PW));
                }
                uint32_t xfa[PB][TAP ? 1 : 3];
#pragma unroll
                for (int a = 0; a < PB; ++a) {
                    const int r = (wave_m * PB + a) * 32 + (lane & 31), cs = TAP ? r : row_cs[r] - 1;
#pragma unroll
                    for (int t = 0; t < (TAP ? 1 : 3); ++t) {
                        const int sl = cs + t;
                        xfa[a][t] = (uint32_t)sl * 128u + (uint32_t)(((lane >> 5) * HALF) ^ FC_SWZ(sl)) * 16u;
                    }
                }
                f32x16_t acc[PB][CB];
#pragma unroll
                for (int b = 0; b < CB; ++b)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int co = co0 + wave_n * (CB * 32) + b * 32 + q * 8 + (lane >> 5) * 4;
                        const float4 bq = (bias && co < g.c_out) ? *reinterpret_cast<const float4 *>(bias + co) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                        for (int a = 0; a < PB; ++a) {
                            acc[a][b][q * 4 + 0] = bq.x;
                            acc[a][b][q * 4 + 1] = bq.y;
                            acc[a][b][q * 4 + 2] = bq.z;
                            acc[a][b][q * 4 + 3] = bq.w;
                        }
                    }
                int xkh = 0, xcc = 0, xkw = 0, xleft = TAP ? 3 * groups : groups;
                uint32_t ld_sx = 0, ld_sel = 0;
                auto next_x = [&]() __attribute__((always_inline)) {
                    ld_sx = xleft > 0 ? (uint32_t)(((xkh * g.dh) * g.w + xkw) * g.c_in + xcc * TK) * (uint32_t)ES : 0u;
                    ld_sel = xleft > 0 ? 1u << (TAP ? xkh * 3 + xkw : xkh) : 0u;
                    --xleft;
                    const int w3 = !TAP || xkw == 2, wrap = w3 & (xcc + 1 == cchunks);
                    if constexpr (TAP) xkw = w3 ? 0 : xkw + 1;
                    xcc = w3 ? (wrap ? 0 : xcc + 1) : xcc;
                    xkh += wrap;
                };
                auto issue_x = [&](int j, uint32_t buf) __attribute__((always_inline)) {
                    if (WHOLE || j < nxl)
                        dma_load16_any(rsrc_x, (hxbits[j / PW] & (ld_sel << (NG * (j % PW)))) ? hxoff[j] : kOutOfRange, ld_sx, lds_wave + buf * XB + (uint32_t)j * (RPL * 128u));
                };
                // Zero stores of a stage: wave v clears the positions of its own label words, in whole 64-piece runs.  A run is one store
                // instruction (a lane with nothing to clear is out of range), so that the waits can count them: z1 and z2 are those of the
                // last two stages.  Lane i holds label word i (an LDS read here would wait for all fragments on their way).
                const int zruns = ((zl + NT - 1) / NT) * cpr, zstep = (zruns + 3 * groups - 1) / (3 * groups);
                const u32x4_t rsrc_z = make_rsrc_words(out + (int64_t)z0 * g.c_out, (uint32_t)zl * (uint32_t)cpr * 16u);
                const uint64_t dropped = drop[min(lane, kWideWords - 1) * kWideWaves + wave];
                int zc = 0, z1 = 0, z2 = 0;
                auto clear_some = [&]() __attribute__((always_inline)) {
                    z2 = z1;
                    z1 = 0;
                    for (int e = 0; e < zstep && zc < zruns; ++e, ++zc) {
                        const int wd = (int)fast_div((uint32_t)zc, wa.cpr), run = zc - wd * cpr; // word, run of 64 pieces in it
                        const uint64_t d = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)dropped, wd) |
                                           (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(dropped >> 32), wd) << 32;
                        if (d == 0) continue;
                        const uint32_t pc = (uint32_t)(run * 64 + lane), ps = fast_div(pc, wa.cpr);
                        store16_zero_nt(rsrc_z, ((d >> ps) & 1ull) ? ((uint32_t)((wd * kWideWaves + wave) * 64 * cpr) + pc) * 16u : kOutOfRange);
                        ++z1;
                    }
                };

#pragma unroll
                for (int d = 0; d < (TAP ? R : 1); ++d) {
                    next_x();
#pragma unroll
                    for (int j = 0; j < XL; ++j) issue_x(j, (uint32_t)d);
                }
                if constexpr (R == 3) { // (nobody needs it before the second barrier)
                    next_w();
#pragma unroll
                    for (int j = 0; j < WL; ++j) issue_w(j, 2);
                }
                wait_vmcnt<(R - 2) * WL>();
                __syncthreads();

                Frag<DT> wf[2][CB], xf[2][PB];
                constexpr int NM = PB * CB, NR = PB + CB; // products and fragment reads of a k-step
                // fragment r of a k-step, in the order the products need them: w0, x0, w1, x1 ..
                auto read_frag = [&](int r, int set, uint32_t xb, uint32_t wb, int t, int kk) __attribute__((always_inline)) {
                    const unsigned char *xs = smem_raw + xb * XB;
                    const unsigned char *ws = smem_raw + W0 + (wb < 2 ? wb * WB : 0u - WB) + (uint32_t)(wave_n * (CB * 32)) * 128u + frag_row;
                    if (r == 1 || r > CB) {
                        const int a = r == 1 ? 0 : r - CB;
                        // (the exclusive or stays here: kept for all k-steps the addresses take the registers of the fragments)
                        uint32_t o = xfa[a][TAP ? 0 : t];
                        if (kk > 0) __asm__ volatile("v_xor_b32 %0, %1, %0" : "+v"(o) : "n"(kk * (int)KSTEP));
                        xf[set][a].load(xs, o);
                    } else {
                        const int b = r == 0 ? 0 : r - 1;
                        wf[set][b].load(ws + b * 4096, ((uint32_t)kk * KSTEP) ^ frag_t16);
                    }
                };
#pragma unroll
                for (int r = 0; r < NR; ++r) read_frag(r, 0, 0, 0, 0, 0);
                // A stage.  Everything that is not a product goes out between two of them, one piece at a time: a product
                // keeps the matrix pipe busy for 32 cycles (8-bit: 64) in which the wave can issue something else, while a burst
                // leaves the pipe idle for its length.
                auto stage = [&](auto xb_c, auto wb_c, auto t_c) __attribute__((always_inline)) {
                    constexpr uint32_t CX = decltype(xb_c)::value, CW = decltype(wb_c)::value;
                    constexpr int t = decltype(t_c)::value;
                    steps<KK>([&](auto kk_c) __attribute__((always_inline)) {
                        constexpr int kk = decltype(kk_c)::value;
                        constexpr bool last = kk == KK - 1;
                        constexpr int BAR = NM / 4; // the barrier of a stage stands after this many products of its last k-step
                        constexpr int from = last ? BAR : 0, gaps = NM - from;
                        // loads: after the barrier the slab R stages ahead, and tap by tap the rows, into the buffers just read;
                        // a line goes out a group ahead, when everyone has left the line before it: with two slabs
                        // on tap 1, in front of which only a slab was sent for, with three on tap 0
                        constexpr int nw = last ? WL : 0, nx = (TAP ? last : t == (R == 3 ? 0 : 1) && kk == 0) ? XL : 0, nl = nw + nx;
                        if constexpr (!TAP && nx > 0) next_x();
                        steps<NM>([&](auto i_c) __attribute__((always_inline)) {
                            constexpr int i = decltype(i_c)::value;
                            if constexpr (last && i == BAR) {
                                // the next stage's slab and rows have landed (what was sent for after them may be on its way, zero
                                // stores included); everyone has read this stage
                                constexpr bool line = !TAP && (R == 3 ? t < 2 : t == 1), counted = line && !WHOLE;
                                constexpr int younger = TAP ? (R - 2) * (WL + XL) : (R == 3 ? WL : 0) + (line && WHOLE ? XL : 0);
                                if (counted || z1 + z2 > 0)
                                    wait_vmcnt_upto16(younger + (counted ? nxl : 0) + z1 + (R == 3 ? z2 : 0));
                                else
                                    wait_vmcnt<younger>();
                                __syncthreads();
                                next_w();
                                if constexpr (TAP) next_x();
                            }
                            acc[i / CB][i % CB] = mfma32<DT>(wf[kk & 1][i % CB], xf[kk & 1][i / CB], acc[i / CB][i % CB]);
                            __builtin_amdgcn_sched_barrier(0);
                            if constexpr (i >= from) {
                                constexpr int j = i - from; // this gap's share of the reads and loads
                                steps<((j + 1) * NR + gaps - 1) / gaps - (j * NR + gaps - 1) / gaps>([&](auto e_c) __attribute__((always_inline)) {
                                    constexpr int r = (j * NR + gaps - 1) / gaps + decltype(e_c)::value;
                                    if constexpr (r < NR) {
                                        if constexpr (last) read_frag(r, 0, TAP ? (CW + 1u) % R : (t == 2 ? CX ^ 1u : CX), (CW + 1u) % R, (t + 1) % 3, 0);
                                        else read_frag(r, (kk + 1) & 1, CX, CW, t, kk + 1);
                                    }
                                });
                                steps<((j + 1) * nl) / gaps - (j * nl) / gaps>([&](auto e_c) __attribute__((always_inline)) {
                                    constexpr int ld = (j * nl) / gaps + decltype(e_c)::value;
                                    if constexpr (ld < nw) issue_w(ld, CW);
                                    else issue_x(ld - nw, TAP ? CW : CX ^ 1u);
                                });
                                __builtin_amdgcn_sched_barrier(0);
                            }
                        });
                        if constexpr (last) clear_some();
                    });
                };
                using I0 = std::integral_constant<uint32_t, 0>;
                using I1 = std::integral_constant<uint32_t, 1>;
                using I2 = std::integral_constant<uint32_t, 2>;
                using T0 = std::integral_constant<int, 0>;
                using T1 = std::integral_constant<int, 1>;
                using T2 = std::integral_constant<int, 2>;
                if constexpr (TAP && R == 3) {
                    for (int gi = 0; gi < groups; ++gi) {
                        stage(I0{}, I0{}, T0{});
                        stage(I1{}, I1{}, T1{});
                        stage(I2{}, I2{}, T2{});
                    }
                } else if constexpr (TAP) {
                    for (int st = 0; st < 3 * groups; st += 2) {
                        stage(I0{}, I0{}, T0{});
                        if (st + 1 < 3 * groups) stage(I1{}, I1{}, T1{});
                    }
                } else {
                    constexpr uint32_t A = R == 3 ? 0 : 1; // (two slabs: the second group starts with the other one)
                    for (int gi = 0; gi < groups; gi += 2) {
                        stage(I0{}, I0{}, T0{});
                        stage(I0{}, I1{}, T1{});
                        stage(I0{}, std::integral_constant<uint32_t, R == 3 ? 2 : 0>{}, T2{});
                        if (gi + 1 < groups) {
                            stage(I1{}, std::integral_constant<uint32_t, A>{}, T0{});
                            stage(I1{}, std::integral_constant<uint32_t, 1 - A>{}, T1{});
                            stage(I1{}, std::integral_constant<uint32_t, R == 3 ? 2 : 1>{}, T2{});
                        }
                    }
                }

                // ---- epilogue: one rounding, ReLU; every wave transposes its blocks of 32 rows x 64 channels through
                // LDS of its own and stores 16 contiguous bytes a lane ----
                wait_vmcnt<0>();
                __syncthreads();
                constexpr int OP = CB * 32 * (int)sizeof(TO) + 16, PPR = CB * 32 * (int)sizeof(TO) / 16, RPI = 64 / PPR, EPT = 16 / (int)sizeof(TO);
                unsigned char *const Os = smem_raw + wave * (32 * OP);
                const int lane = thread_number() & 63;
                const int pc = lane % PPR, rr = lane / PPR;
                const int co = co0 + wave_n * (CB * 32) + pc * EPT;
#pragma unroll
                for (int a = 0; a < PB; ++a) {
#pragma unroll
                    for (int b = 0; b < CB; ++b)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const int cl = b * 32 + q * 8 + (lane >> 5) * 4;
                            float v0 = acc[a][b][q * 4 + 0], v1 = acc[a][b][q * 4 + 1];
                            float v2 = acc[a][b][q * 4 + 2], v3 = acc[a][b][q * 4 + 3];
                            if constexpr (sizeof(TO) == 4) {
                                if (g.flags & FC_RELU) {
                                    v0 = relu_keep_nan(v0); v1 = relu_keep_nan(v1);
                                    v2 = relu_keep_nan(v2); v3 = relu_keep_nan(v3);
                                }
                                store4<ODT, TO>(reinterpret_cast<TO *>(Os + (lane & 31) * OP) + cl, v0, v1, v2, v3);
                            } else if constexpr (sizeof(TO) == 1) {
                                uint32_t pk;
                                store4<ODT, TO>(reinterpret_cast<TO *>(&pk), v0, v1, v2, v3);
                                if (g.flags & FC_RELU) pk = relu_packed8(pk);
                                *reinterpret_cast<uint32_t *>(Os + (lane & 31) * OP + cl) = pk;
                            } else {
                                uint2 pk;
                                store4<ODT, TO>(reinterpret_cast<TO *>(&pk), v0, v1, v2, v3);
                                if (g.flags & FC_RELU) {
                                    pk.x = relu_packed16(pk.x);
                                    pk.y = relu_packed16(pk.y);
                                }
                                *reinterpret_cast<uint2 *>(Os + (lane & 31) * OP + cl * 2) = pk;
                            }
                        }
                    __asm__ volatile("" ::: "memory");
                    u32x4_t pv[32 / RPI];
                    int pp[32 / RPI];
#pragma unroll
                    for (int i = 0; i < 32 / RPI; ++i) {
                        const int r = rr + i * RPI;
                        pp[i] = row_p[(wave_m * PB + a) * 32 + r];
                        pv[i] = *reinterpret_cast<const u32x4_t *>(Os + r * OP + pc * 16);
                    }
#pragma unroll
                    for (int i = 0; i < 32 / RPI; ++i)
                        if (pp[i] >= 0 && co < g.c_out)
                            __builtin_nontemporal_store(pv[i], reinterpret_cast<u32x4_t *>(out + (int64_t)pp[i] * g.c_out + co));
                    __asm__ volatile("" ::: "memory");
                }
            };
            auto run_form = [&](auto tap_c) __attribute__((always_inline)) {
                switch (k) {
                case 1: run(std::integral_constant<int, 1>{}, tap_c); break;
                case 2: run(std::integral_constant<int, 2>{}, tap_c); break;
                case 3: run(std::integral_constant<int, 3>{}, tap_c); break;
                default: if constexpr (PBX >= 4) run(std::integral_constant<int, 4>{}, tap_c); break;
                }
            };
            if (by_tap) run_form(std::true_type{}); else run_form(std::false_type{});
            g0 += k;
        }
    }
    if (zero_fill && !clear_in_loop)
        clear_irrelevant_runs(g, mask_in, mask_out, out, cpr, wa.cpr, zt0, zx1, slot_x * kWideWaves + wave, per_xcd * kWideWaves);
}

// ---------------------------------------------------------------------------

#if !defined(FC_WIDE_PART) || FC_WIDE_PART == 0
bool conv_wide_supported(const Geom &g, int in_dtype, int out_dtype)
{
    if (in_dtype != FC_BF16 && in_dtype != FC_F16 && in_dtype != FC_FP8) return false;
    if (out_dtype != (in_dtype == FC_FP8 ? FC_BF16 : in_dtype) && out_dtype != FC_F32 && out_dtype != FC_FP8) return false;
    const int es = in_dtype == FC_FP8 ? 1 : 2;
    if (!(g.kh == 3 && g.kw == 3 && g.sw == 1 && g.dw == 1) || g.c_out % 128 != 0) return false;
    if ((g.c_in * es) % 128 != 0) return false; // whole chunks
    return !(g.flags & FC_COMPACT_IN);
}
#endif

template <int DT, typename TO, int WM, int PBX, int SL, int SLS>
static hipError_t launch_wide(const Geom &g, int grid, const void *x, const uint8_t *mask_in, const uint8_t *mask_out, const void *w,
                              const float *bias, const int32_t *idx, const int32_t *count, void *out, hipStream_t s)
{
    constexpr int TN = (kWideWaves / WM) * 64;
    auto kern = k_conv_wide<DT, TO, WM, PBX, SL, SLS>;
    constexpr size_t lds = wide_lds_bytes<WM, TN, PBX, SL, SLS>();
    static_assert(lds <= 160 * 1024, "LDS of a CU");
    // the dynamic LDS limit is raised once per function and device
    static std::atomic<uint64_t> attr_devices{0};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t dev_bit = 1ull << (dev & 63);
    if (!(attr_devices.load(std::memory_order_acquire) & dev_bit)) {
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attr_devices.fetch_or(dev_bit, std::memory_order_release);
    }
    WideArgs wa;
    wa.n_nt = (g.c_out + TN - 1) / TN;
    wa.cpr = make_fastdiv((uint32_t)g.c_out * (uint32_t)sizeof(TO) / 16u);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kWideThreads), lds, s, g, wa, (const unsigned char *)x, mask_in, mask_out,
                       (const unsigned char *)w, bias, idx, count, (TO *)out);
    return hipGetLastError();
}

template <int DT, typename TO>
static hipError_t launch_wide_shape(const Geom &g, int grid, const void *x, const uint8_t *mask_in, const uint8_t *mask_out,
                                    const void *w, const float *bias, const int32_t *idx, const int32_t *count, void *out, hipStream_t s)
{
    // (8-bit fragments are twice as large: three blocks a wave, or the loop spills)
    if (g.c_out % 256 == 0) return launch_wide<DT, TO, 2, DT == FC_FP8 ? 3 : 4, DT == FC_FP8 ? 256 : 320, 192>(g, grid, x, mask_in, mask_out, w, bias, idx, count, out, s);
    return launch_wide<DT, TO, 4, 3, 448, 0>(g, grid, x, mask_in, mask_out, w, bias, idx, count, out, s);
}

// The instances are spread over nine translation units, one per pair of types (-DFC_WIDE_PART=p; without the macro this file
// is one unit that holds everything); part 0 also holds the entry points.
#define FC_WIDE_PARAMS                                                                                                   \
    const Geom &g, int grid, const void *x, const uint8_t *mask_in, const uint8_t *mask_out, const void *w, const float *bias, \
        const int32_t *idx, const int32_t *count, void *out, hipStream_t s
#ifndef FC_WIDE_PART
#define FC_WIDE_PART -1
#endif
#define FC_WIDE_UNIT(p, name, DT, TO) hipError_t name(FC_WIDE_PARAMS);
#define FC_WIDE_UNITS                                      \
    FC_WIDE_UNIT(0, launch_wide_bf16, FC_BF16, uint16_t)   \
    FC_WIDE_UNIT(1, launch_wide_bf16_f32, FC_BF16, float)  \
    FC_WIDE_UNIT(2, launch_wide_bf16_fp8, FC_BF16, uint8_t) \
    FC_WIDE_UNIT(3, launch_wide_f16, FC_F16, uint16_t)     \
    FC_WIDE_UNIT(4, launch_wide_f16_f32, FC_F16, float)    \
    FC_WIDE_UNIT(5, launch_wide_f16_fp8, FC_F16, uint8_t)  \
    FC_WIDE_UNIT(6, launch_wide_fp8_bf16, FC_FP8, uint16_t) \
    FC_WIDE_UNIT(7, launch_wide_fp8_f32, FC_FP8, float)    \
    FC_WIDE_UNIT(8, launch_wide_fp8, FC_FP8, uint8_t)
FC_WIDE_UNITS
#undef FC_WIDE_UNIT
// (a unit's definition: the instances of its pair of types)
#define FC_WIDE_DEFINE(name, DT, TO) \
    hipError_t name(FC_WIDE_PARAMS) { return launch_wide_shape<DT, TO>(g, grid, x, mask_in, mask_out, w, bias, idx, count, out, s); }
#define FC_IN_PART(p) (FC_WIDE_PART < 0 || FC_WIDE_PART == (p))
#if FC_IN_PART(0)
FC_WIDE_DEFINE(launch_wide_bf16, FC_BF16, uint16_t)
#endif
#if FC_IN_PART(1)
FC_WIDE_DEFINE(launch_wide_bf16_f32, FC_BF16, float)
#endif
#if FC_IN_PART(2)
FC_WIDE_DEFINE(launch_wide_bf16_fp8, FC_BF16, uint8_t)
#endif
#if FC_IN_PART(3)
FC_WIDE_DEFINE(launch_wide_f16, FC_F16, uint16_t)
#endif
#if FC_IN_PART(4)
FC_WIDE_DEFINE(launch_wide_f16_f32, FC_F16, float)
#endif
#if FC_IN_PART(5)
FC_WIDE_DEFINE(launch_wide_f16_fp8, FC_F16, uint8_t)
#endif
#if FC_IN_PART(6)
FC_WIDE_DEFINE(launch_wide_fp8_bf16, FC_FP8, uint16_t)
#endif
#if FC_IN_PART(7)
FC_WIDE_DEFINE(launch_wide_fp8_f32, FC_FP8, float)
#endif
#if FC_IN_PART(8)
FC_WIDE_DEFINE(launch_wide_fp8, FC_FP8, uint8_t)
#endif

#if FC_IN_PART(0)
hipError_t launch_conv_wide(const Geom &g, int in_dtype, int out_dtype, int grid, const void *x, const uint8_t *mask_in,
                            const uint8_t *mask_out, const void *w, const float *bias, const int32_t *idx, const int32_t *count,
                            void *out, hipStream_t s)
{
    using Launch = hipError_t (*)(FC_WIDE_PARAMS);
    static const Launch by_types[3][3] = {{launch_wide_bf16, launch_wide_bf16_f32, launch_wide_bf16_fp8},
                                          {launch_wide_f16, launch_wide_f16_f32, launch_wide_f16_fp8},
                                          {launch_wide_fp8_bf16, launch_wide_fp8_f32, launch_wide_fp8}};
    const int in = in_dtype == FC_BF16 ? 0 : (in_dtype == FC_F16 ? 1 : 2);
    const int to = out_dtype == FC_F32 ? 1 : (out_dtype == FC_FP8 ? 2 : 0);
    return by_types[in][to](g, grid, x, mask_in, mask_out, w, bias, idx, count, out, s);
}
#endif

} // namespace fc
