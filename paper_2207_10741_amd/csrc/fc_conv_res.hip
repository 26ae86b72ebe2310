// Focused 3x3 convolution of 128-byte pixels (64 channels of a 16-bit type, 128 of the 8-bit one) into slices of
// 64 output channels, with the nine taps' weights resident in LDS (Sec. III-A: a GEMM over the kept patches
// only, with the dense layer's weights).
//
// One workgroup per CU keeps its slice's weights (72 KB) in LDS for the whole launch; eight of its waves are
// pipelines of their own over blocks of 32 kept rows, as in the 1x1 kernel next door.  Bound: LDS reads (1.5 KB a matrix
// instruction) and the vector instructions of a block's set-up beside them; memory where the rows are cleared too.
// What the tap-by-tap form of the 1x1 kernel, which ran these layers before, spent its time on was the chain of round
// trips (one gather of 4 KB in flight a wave, nine a block) and reading a pixel from memory once per kernel row.
//
// - Pixel line (unit horizontal stride and dilation): along a run of horizontally adjacent kept positions the
//   left pixel of one is the centre pixel of the one before, so a block lays the pixels under a kernel row
//   out on a line of slots - one per row, one more at either end of every run - and gathers it once for the three
//   horizontal taps: three gathers of up to 40 pixels instead of nine of 32.  A block that needs more slots (a
//   fragmented mask) goes tap by tap.
// - Blocks are dealt to the waves of an XCD side by side, so that the rows above and below pass through its L2 together.
// - Zero-fill by waves of its own: four more waves of the workgroup do nothing but clear irrelevant rows while the
//   eight multiply; their stores share no counter with anybody's gathers.
// - Fragments are read two steps ahead of their products, and what follows from the lane number is computed where it is
//   used instead of kept: 141 registers, no spills at three waves per SIMD.
//
// 64 -> 64 channels, bf16, on 8 x 1080 x 1920, half kept (us; tap by tap -> lines -> and fragments ahead -> and blocks side by
// side): zero-filled 1 204 -> 1 003 -> 994 -> 820, chained 1 010 -> 877 -> 826 -> 742; 32 x 120 x 160, 48 % irrelevant, zero-filled
// 44.6 -> 33.7.  Salt-and-pepper masks of half the pixels, chained, 32 x 120 x 160: 38.9 -> 44 on inputs in the caches already,
// 50 either way on others.
//
// A slot is gated per kernel row (inside the image and relevant); the mask bytes under a block's slots are
// fetched into LDS a block ahead, and what a lane must not read is sent out of range (zeros, no memory access).
#include "fc_dma_util.hpp"
#include <atomic>
#include <type_traits>

namespace fc {

constexpr int kResWaves = 8;                                   // waves that multiply
constexpr int kResClearWaves = 4;                              // waves that clear irrelevant rows
constexpr int kResSlots = 40;                                  // slots of a pixel line
constexpr uint32_t kResLineBytes = kResSlots * 128u;
constexpr uint32_t kResWeightBytes = 9u * 64u * 128u;
// of a wave: two lines, the list entries of a unit (one dword per lane), the mask bytes under its slots (two dwords per
// lane: kernel row * 40 + slot), the slot table
constexpr uint32_t kResWaveBytes = 2u * kResLineBytes + 256u + 512u + kResSlots * 4u;
constexpr uint32_t kResLdsBytes = kResWeightBytes + 512u + kResWaves * kResWaveBytes;
static_assert(kResLdsBytes <= 160u * 1024u, "LDS of a CU");

// DT: storage type; TO: float or the 16-bit / 8-bit carrier of the output; bias_last: the bias is added to the finished sum
// (else the sum starts from it).
template <int DT, typename TO>
__global__ __launch_bounds__((kResWaves + kResClearWaves) * 64, 1)
void k_conv_res3(Geom g, FastDiv div_cpr, bool bias_last, const unsigned char *__restrict__ x, const uint8_t *__restrict__ mask_in,
                 const uint8_t *__restrict__ mask_out, const unsigned char *__restrict__ w, const float *__restrict__ bias,
                 const int32_t *__restrict__ idx, const int32_t *__restrict__ count, TO *__restrict__ out)
{
    constexpr int ODT = DT == FC_FP8 ? FC_BF16 : DT;    // 16-bit output format
    constexpr uint32_t KSTEP = kStepBytes<DT>;
    constexpr int KK = 128 / (int)KSTEP;                // matrix instructions per tap and block
    constexpr int LS = kResSlots, LJ = LS / 8;          // wave loads of a line (eight slots each)

    extern __shared__ __align__(16) unsigned char smem_raw[];
    const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>(smem_raw);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nwaves = (int)blockDim.x >> 6;
    const int l32 = lane & 31, half = lane >> 5;
    const float *bias_s = reinterpret_cast<const float *>(smem_raw + kResWeightBytes);
    const bool packed_masks = (g.flags & FC_PACKED_MASKS) != 0;
    const bool compact_out = (g.flags & FC_COMPACT_OUT) != 0;
    int rows = g.m;
    if (idx) rows = *count;
    rows = __builtin_amdgcn_readfirstlane(rows);

    // slices, groups and shares as in the 1x1 kernel: the workgroups of an XCD form groups of n_slices neighbours
    // that share their rows, XCD j takes the j-th contiguous eighth of the rows
    const int n_slices = (g.c_out + 63) / 64;
    const int in_xcd = (int)blockIdx.x >> 3, groups_per_xcd = ((int)gridDim.x >> 3) / n_slices;
    const bool spare = in_xcd >= groups_per_xcd * n_slices;
    const int co0 = spare ? 0 : (in_xcd % n_slices) * 64;
    const int co_left = g.c_out - co0;
    // (an output larger than the memory-side cache is streamed past it, as in the 1x1 kernel)
    const bool stream_out = (int64_t)rows * g.c_out * (int)sizeof(TO) > (256ll << 20);

    // ---- the weights: LDS row (tap, output channel), 16-byte pieces swizzled by the channel ----
    if (!spare) {
        const u32x4_t rsrc_w = make_rsrc_words(w, (uint32_t)g.c_out * 9u * 128u);
        for (int ii = wave; ii < 72; ii += nwaves) {
            const int tap = ii >> 3, co = (ii & 7) * 8 + (lane >> 3);
            const uint32_t off = (uint32_t)(co0 + co) * (9u * 128u) + (uint32_t)tap * 128u + (uint32_t)((lane & 7) ^ (int)FC_SWZ(co)) * 16u;
            dma_load16(rsrc_w, co < co_left ? off : kOutOfRange, lds0 + (uint32_t)ii * 1024u);
        }
        // what the sums start from, and what is added to them at the end: the bias in one of the two, zeros in the other
        const u32x4_t rsrc_b = make_rsrc_words(bias, bias ? (uint32_t)g.c_out * 4u : 0u);
        if (wave == 0) {
            dma_load4(rsrc_b, bias_last ? kOutOfRange : (uint32_t)(co0 + lane) * 4u, lds0 + kResWeightBytes);
            dma_load4(rsrc_b, bias_last ? (uint32_t)(co0 + lane) * 4u : kOutOfRange, lds0 + kResWeightBytes + 256u);
        }
    }

    // ---- the waves that clear ----
    if (wave >= kResWaves) {
        wait_vmcnt<0>();
        __syncthreads();
        const int per_wg = nwaves - kResWaves;
        clear_irrelevant_runs(g, mask_in, mask_out, out, g.c_out * (int)sizeof(TO) / 16, div_cpr, 0, g.m,
                              (int)blockIdx.x * per_wg + (wave - kResWaves), (int)gridDim.x * per_wg);
        return;
    }

    unsigned char *const my = smem_raw + kResWeightBytes + 512u + (size_t)wave * kResWaveBytes;
    const uint32_t my0 = lds0 + kResWeightBytes + 512u + (uint32_t)wave * kResWaveBytes;
    const int32_t *const idx_w = reinterpret_cast<const int32_t *>(my + 2 * kResLineBytes);
    const uint32_t *const mask_w = reinterpret_cast<const uint32_t *>(my + 2 * kResLineBytes + 256u);
    uint32_t *const tab = reinterpret_cast<uint32_t *>(my + 2 * kResLineBytes + 768u);
    const uint32_t idx0 = my0 + 2 * kResLineBytes, mask0 = idx0 + 256u, tap0 = my0 + 4096u;

    // The kept rows in blocks of 32: XCD j takes the j-th contiguous eighth, and its waves take neighbouring blocks
    // side by side, so that the image rows above and below a block's pass through the XCD's L2 at about the same
    // time.  (As contiguous runs, one a wave, a pixel came from memory once per kernel row: 64 -> 64 on 8 x 1080 x 1920, half
    // kept, 826 us at 5.4 TB/s.)
    const int nb = (rows + 31) >> 5, xcd = (int)blockIdx.x & 7;
    const int blk_step = groups_per_xcd * kResWaves;
    const int blk_end = (int)(((int64_t)nb * (xcd + 1)) >> 3);
    int blk = (int)(((int64_t)nb * xcd) >> 3) + (in_xcd / n_slices) * kResWaves + wave; // the block units are taken from
    if (spare) blk = blk_end;

    const u32x4_t rsrc_x = make_rsrc_words(x, (uint32_t)g.n * g.h * g.w * 128u);
    const u32x4_t rsrc_i = make_rsrc_words(idx, (uint32_t)rows * 4u);
    const u32x4_t rsrc_m = make_rsrc_words(mask_in, packed_masks ? (uint32_t)(((int64_t)g.n * g.h * g.w + 7) >> 3)
                                                                 : (uint32_t)g.n * g.h * g.w);
    const uint32_t krow_pix = (uint32_t)(g.dh * g.w); // pixels from one kernel row to the next

    // loads issued so far by this wave, and that count right after the last load of what is awaited
    int issued = 0, mark_idx = 0, mark_m = 0, mark_t = 0, mark_x = 0;

    auto issue_idx = [&]() __attribute__((always_inline)) { // of block `blk`
        if (!idx) return;
        lds_reads_done();
        dma_load4(rsrc_i, lane < 32 ? (uint32_t)(blk * 32 + lane) * 4u : kOutOfRange, idx0);
        issued += 1;
        mark_idx = issued;
    };

    // The unit of block `blk`, from its list entries (blk then moves on): where its rows go, the centre slot of every
    // row, and the slot table: the pixel under kernel row 0 (its low 25 bits: pixels are 128 bytes of a tensor below
    // 2^32 bytes) and, bits 28 .. 30, the kernel rows that lie inside the image.  The mask bytes under the slots
    // are sent for.  Rows that need more than LS slots go tap by tap: n_w0 is then a row's nine taps that are read,
    // n_w1 the pixel under its first tap.
    constexpr uint32_t kPixBits = 0x1ffffffu;
    int n_p = -1, n_cs = 1;
    bool n_frag = false, n_lds = false, c_frag = false; // (c_: the current unit)
    uint32_t n_w0 = 0, n_w1 = 0; // slot words of this lane's (kernel row, slot) pairs `lane` and 64 + lane
    // (what follows from the lane number alone is computed where it is used: kept for the whole loop it takes the
    // registers of the fragments)
    auto own_lane = [&]() __attribute__((always_inline)) {
        int v = lane;
        __asm__ volatile("" : "+v"(v));
        return v;
    };
    auto presetup = [&]() __attribute__((always_inline)) {
        const int lane = own_lane(), l32 = lane & 31, half = lane >> 5;
        const int pair1 = lane + 64;
        const int kh0 = lane >= LS ? 1 : 0, kh1 = pair1 >= 2 * LS ? 2 : 1;
        const int sl0 = lane - kh0 * LS, sl1 = min(pair1 - kh1 * LS, LS - 1);
        const bool live1 = pair1 < 3 * LS;
        const int r = blk * 32 + l32;
        const bool valid = r < rows;
        int p = r;
        if (idx) {
            wait_vmcnt_upto(issued - mark_idx);
            p = idx_w[l32];
        }
        p = valid ? p : -1;
        const int prev = __shfl(p, (lane & 32) | ((l32 + 31) & 31), 64), next = __shfl(p, (lane & 32) | ((l32 + 1) & 31), 64);
        const int q1 = (int)fast_div((uint32_t)(valid ? p : 0), g.div_wo);
        const int ow = (valid ? p : 0) - q1 * g.wo;
        const int n = (int)fast_div((uint32_t)q1, g.div_ho);
        const int oh = q1 - n * g.ho;
        const bool ladj = valid && l32 > 0 && prev == p - 1 && ow > 0;
        const bool radj = valid && l32 < 31 && next == p + 1 && ow < g.wo - 1;
        const int cnt = valid ? 1 + !ladj + !radj : 0;
        int incl = wave_inclusive_scan(cnt);
        const int lower = __builtin_amdgcn_readlane(incl, 31);
        incl -= half ? lower : 0; // (both halves hold the same rows)
        const int cs = incl - cnt + !ladj;
        const int ih0 = oh * g.sh - g.ph, iwc = ow - g.pw + 1;
        const uint32_t pix = (uint32_t)((n * g.h + ih0) * g.w + iwc);
        n_frag = lower > LS;
        n_p = valid ? (compact_out ? r : p) : -1;
        n_cs = valid ? cs : 1;
        blk += blk_step;
        uint32_t w0, w1;
        if (!n_frag) {
            uint32_t rows_in = 0;
#pragma unroll
            for (int k = 0; k < 3; ++k) rows_in |= (uint32_t)((uint32_t)(ih0 + k * g.dh) < (uint32_t)g.h) << (28 + k);
            if (lane < LS) tab[lane] = 0;
            wave_lds_order(); // (lanes write entries of one another)
            if (valid && half == 0) {
                tab[cs] = (pix & kPixBits) | ((uint32_t)iwc < (uint32_t)g.w ? rows_in : 0u);
                if (!ladj) tab[cs - 1] = ((pix - 1u) & kPixBits) | ((uint32_t)(iwc - 1) < (uint32_t)g.w ? rows_in : 0u);
                if (!radj) tab[cs + 1] = ((pix + 1u) & kPixBits) | ((uint32_t)(iwc + 1) < (uint32_t)g.w ? rows_in : 0u);
            }
            wave_lds_order(); // (lanes write entries of one another)
            w0 = tab[sl0];
            w1 = live1 ? tab[sl1] : 0u;
            if (mask_in) {
                const uint32_t px0 = (w0 + (uint32_t)kh0 * krow_pix) & kPixBits, px1 = (w1 + (uint32_t)kh1 * krow_pix) & kPixBits;
                lds_reads_done();
                dma_load1(rsrc_m, ((w0 >> (28 + kh0)) & 1u) ? (packed_masks ? px0 >> 3 : px0) : kOutOfRange, mask0);
                dma_load1(rsrc_m, ((w1 >> (28 + kh1)) & 1u) ? (packed_masks ? px1 >> 3 : px1) : kOutOfRange, mask0 + 256u);
                issued += 2;
                mark_m = issued;
            }
        } else {
            // Taps 2q + half of row l32.  While the current unit goes tap by tap as well, the last 1 KB of either buffer is
            // free and takes the mask bytes; else they are loaded plainly (waiting for them drains the gathers in
            // flight, one stage in nine).
            const bool to_lds = mask_in && c_frag;
            uint32_t bits = 0;
#pragma unroll
            for (int q = 0; q < 5; ++q) {
                const int t = 2 * q + half, kh = (t * 11) >> 5, kw = t - kh * 3; // t / 3 for t < 10
                const int ih = ih0 + kh * g.dh, iw = iwc - 1 + kw;
                const bool in = valid && t < 9 && (uint32_t)ih < (uint32_t)g.h && (uint32_t)iw < (uint32_t)g.w;
                const uint32_t px = in ? (uint32_t)((n * g.h + ih) * g.w + iw) : 0u;
                if (to_lds) {
                    if (q == 0) lds_reads_done();
                    dma_load1(rsrc_m, in ? (packed_masks ? px >> 3 : px) : kOutOfRange, tap0 + (q < 4 ? (uint32_t)q * 256u : kResLineBytes));
                } else {
                    bits |= (uint32_t)(in && (!mask_in || mask_at(mask_in, px, packed_masks))) << t;
                }
            }
            if (to_lds) {
                issued += 5;
                mark_t = issued;
            }
            n_lds = to_lds;
            w0 = bits | (uint32_t)__shfl((int)bits, lane ^ 32, 64);
            w1 = pix - 1u;
        }
        n_w0 = w0;
        n_w1 = w1;
    };

    // What the next unit's gathers read: the offset of slot (tap by tap: row) 8j + lane / 8 under kernel row (tap) 0, and per
    // kernel row the slots that are read (tap by tap: the taps of its four rows, 16 bits each).  Written when the
    // current unit has sent for its last gather.
    uint32_t off[LJ];
    uint64_t read[3] = {0, 0, 0};
    uint64_t val = 0;
    auto setup = [&]() __attribute__((always_inline)) {
        const int lane = own_lane();
        if (!n_frag) {
            const int kh0 = lane >= LS ? 1 : 0, kh1 = lane + 64 >= 2 * LS ? 2 : 1;
            uint32_t ok0 = (n_w0 >> (28 + kh0)) & 1u, ok1 = (n_w1 >> (28 + kh1)) & 1u;
            if (mask_in) {
                wait_vmcnt_upto(issued - mark_m);
                const uint32_t m0 = mask_w[lane], m1 = mask_w[64 + lane];
                const uint32_t px0 = n_w0 + (uint32_t)kh0 * krow_pix, px1 = n_w1 + (uint32_t)kh1 * krow_pix;
                ok0 &= packed_masks ? (m0 >> (px0 & 7u)) & 1u : (uint32_t)(m0 != 0);
                ok1 &= packed_masks ? (m1 >> (px1 & 7u)) & 1u : (uint32_t)(m1 != 0);
            }
            const uint64_t b0 = __ballot(ok0 != 0), b1 = __ballot(ok1 != 0);
            constexpr uint64_t kSlotBits = (1ull << LS) - 1ull;
            read[0] = b0 & kSlotBits;
            read[1] = ((b0 >> LS) | (b1 << (64 - LS))) & kSlotBits;
            read[2] = (b1 >> (2 * LS - 64)) & kSlotBits;
#pragma unroll
            for (int j = 0; j < LJ; ++j) {
                const int sl = j * 8 + (lane >> 3);
                off[j] = (tab[sl] << 7) + (uint32_t)((lane & 7) ^ FC_SWZ(sl)) * 16u;
            }
        } else {
            if (n_lds) {
                wait_vmcnt_upto(issued - mark_t);
                const int half = lane >> 5;
                uint32_t bits = 0;
#pragma unroll
                for (int q = 0; q < 5; ++q) {
                    const int t = 2 * q + half, kh = (t * 11) >> 5, kw = t - kh * 3;
                    const uint32_t m = *reinterpret_cast<const uint32_t *>(my + 4096 + (q < 4 ? q * 256 : (int)kResLineBytes) + lane * 4);
                    const uint32_t px = n_w1 + (uint32_t)kh * krow_pix + (uint32_t)kw;
                    bits |= (packed_masks ? (m >> (px & 7u)) & 1u : (uint32_t)(m != 0)) << t;
                }
                n_w0 = bits | (uint32_t)__shfl((int)bits, lane ^ 32, 64);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int row = j * 8 + (lane >> 3);
                off[j] = ((uint32_t)__shfl((int)n_w1, row, 64) << 7) + (uint32_t)((lane & 7) ^ FC_SWZ(row)) * 16u;
            }
            const int row = lane >> 3;
            val = ((uint64_t)((uint32_t)__shfl((int)n_w0, row + 16, 64) | (uint32_t)__shfl((int)n_w0, row + 24, 64) << 16) << 32) |
                  ((uint32_t)__shfl((int)n_w0, row, 64) | (uint32_t)__shfl((int)n_w0, row + 8, 64) << 16);
        }
    };
    auto issue_line = [&](int kh, uint32_t to) __attribute__((always_inline)) {
        lds_reads_done();
        const uint32_t delta = (uint32_t)kh * krow_pix * 128u, to0 = __builtin_amdgcn_readfirstlane(my0 + to * kResLineBytes);
#pragma unroll
        for (int j = 0; j < LJ; ++j) {
            const uint32_t on = ((uint32_t)(read[kh] >> (8 * j)) >> (lane >> 3)) & 1u;
            dma_load16_s(rsrc_x, on ? off[j] + delta : kOutOfRange, 0u, to0 + (uint32_t)j * 1024u);
        }
        issued += LJ;
        mark_x = issued;
    };
    auto issue_tap = [&](int t, uint32_t to) __attribute__((always_inline)) {
        lds_reads_done();
        const uint32_t kh = (uint32_t)(t * 11) >> 5, delta = (kh * krow_pix + (uint32_t)t - kh * 3u) * 128u;
        const uint32_t to0 = __builtin_amdgcn_readfirstlane(my0 + to * kResLineBytes);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t on = ((uint32_t)(val >> (16 * j)) >> t) & 1u;
            dma_load16_s(rsrc_x, on ? off[j] + delta : kOutOfRange, 0u, to0 + (uint32_t)j * 1024u);
        }
        issued += 4;
        mark_x = issued;
    };

    // fragment addressing as everywhere here: in k-step kk lane reads piece (KSTEP / 16) kk + (lane >> 5) (KSTEP / 32) of its row,
    // stored at slot piece ^ swizzle(row)
    const uint32_t hp = (uint32_t)(half * (int)(KSTEP / 32u));
    const uint32_t wfrag = (uint32_t)l32 * 128u + (hp ^ FC_SWZ(l32)) * 16u;

    bool more = blk < blk_end;
    uint32_t buf = 0;
    if (more) {
        issue_idx();
        presetup();
        if (blk < blk_end) issue_idx();
        setup();
        if (n_frag) issue_tap(0, 0); else issue_line(0, 0);
    }
    wait_vmcnt_upto(issued); // this wave's share of the weights (sent for before everything counted)
    __syncthreads();

    f32x16_t acc[2];
    while (more) {
        const int c_p = n_p, c_cs = n_cs;
        c_frag = n_frag;
        more = blk < blk_end; // a unit after this one
        // (around the first and last gather of a unit: the next unit's rows are looked up, and sent for)
        auto look_ahead = [&]() __attribute__((always_inline)) {
            if (!more) return;
            presetup();
            if (blk < blk_end) issue_idx();
        };
        auto next_unit = [&]() __attribute__((always_inline)) {
            if (!more) return;
            setup();
            if (n_frag) issue_tap(0, buf ^ 1u); else issue_line(0, buf ^ 1u);
        };
        // (set when the next unit has been looked up: that takes registers as well)
        auto start_sums = [&]() __attribute__((always_inline)) {
            const int half = own_lane() >> 5;
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float4 bq = *reinterpret_cast<const float4 *>(bias_s + b * 32 + q * 8 + half * 4);
                    acc[b][q * 4 + 0] = bq.x;
                    acc[b][q * 4 + 1] = bq.y;
                    acc[b][q * 4 + 2] = bq.z;
                    acc[b][q * 4 + 3] = bq.w;
                }
        };
        // Steps of one row fragment and two weight fragments; the fragments of step s + kAhead are read before
        // step s is multiplied, in that order.  (Left to itself the compiler reads a fragment right before its product,
        // and two waves on a SIMD do not hide thirty-six LDS latencies a unit: 1 003 against 994 us zero-filled, 877 against 826
        // us chained, 64 -> 64 on 8 x 1080 x 1920.)
        constexpr int kAhead = DT == FC_FP8 ? 1 : 2;
        Frag<DT> xf[kAhead + 1], wf[kAhead + 1][2];
        auto stage = [&](auto taps_c, const unsigned char *xs, const uint32_t *xfa, const unsigned char *ws0) __attribute__((always_inline)) {
            constexpr int STEPS = decltype(taps_c)::value * KK;
            auto read_step = [&](int st) __attribute__((always_inline)) {
                const int t = st / KK, kk = st - t * KK;
                const unsigned char *ws = ws0 + (uint32_t)t * (64u * 128u);
                xf[st % (kAhead + 1)].load(xs, xfa[t] ^ ((uint32_t)kk * KSTEP));
#pragma unroll
                for (int b = 0; b < 2; ++b) wf[st % (kAhead + 1)][b].load(ws + b * 4096, wfrag ^ ((uint32_t)kk * KSTEP));
            };
#pragma unroll
            for (int st = 0; st < kAhead; ++st) read_step(st);
#pragma unroll
            for (int st = 0; st < STEPS; ++st) {
                if (st + kAhead < STEPS) read_step(st + kAhead);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int b = 0; b < 2; ++b) acc[b] = mfma32<DT>(wf[st % (kAhead + 1)][b], xf[st % (kAhead + 1)], acc[b]);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        // a gather goes out first, into the buffer freed last: the next kernel row's (tap's), or the next unit's first
        if (!c_frag) {
            uint32_t xfa[3];
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                const uint32_t sl = (uint32_t)(c_cs + t - 1);
                xfa[t] = sl * 128u + (hp ^ FC_SWZ(sl)) * 16u;
            }
#pragma unroll
            for (int kh = 0; kh < 3; ++kh) {
                const int mark = mark_x; // (of the line multiplied now)
                if (kh < 2) issue_line(kh + 1, buf ^ 1u);
                if (kh == 0) look_ahead();
                if (kh == 0) start_sums();
                if (kh == 2) next_unit();
                wait_vmcnt_upto(issued - mark);
                stage(std::integral_constant<int, 3>{}, my + buf * kResLineBytes, xfa, smem_raw + (uint32_t)kh * (3u * 64u * 128u));
                buf ^= 1u;
            }
        } else {
            start_sums();
#pragma unroll 1
            for (int t = 0; t < 9; ++t) {
                const int mark = mark_x;
                if (t < 8) issue_tap(t + 1, buf ^ 1u);
                if (t == 0) look_ahead();
                if (t == 8) next_unit();
                wait_vmcnt_upto(issued - mark);
                stage(std::integral_constant<int, 1>{}, my + buf * kResLineBytes, &wfrag, smem_raw + (uint32_t)t * (64u * 128u));
                buf ^= 1u;
            }
        }
        {
            const int lane = own_lane(), l32 = lane & 31, half = lane >> 5;
            unsigned char *const xs = my + (buf ^ 1u) * kResLineBytes; // the buffer multiplied last
            // one rounding; 16- and 8-bit rows leave through the line just consumed (its fragments are in
            // registers, a wave's LDS accesses execute in order) as whole 16-byte pieces
#pragma unroll
            for (int b = 0; b < 2; ++b) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int cl = b * 32 + q * 8 + half * 4; // this lane's four channels of the slice
                    const float4 bq = *reinterpret_cast<const float4 *>(bias_s + 64 + cl);
                    float v0 = acc[b][q * 4] + bq.x, v1 = acc[b][q * 4 + 1] + bq.y;
                    float v2 = acc[b][q * 4 + 2] + bq.z, v3 = acc[b][q * 4 + 3] + bq.w;
                    if constexpr (sizeof(TO) == 4) {
                        if (g.flags & FC_RELU) {
                            v0 = relu_keep_nan(v0); v1 = relu_keep_nan(v1);
                            v2 = relu_keep_nan(v2); v3 = relu_keep_nan(v3);
                        }
                        if (c_p >= 0 && cl < co_left)
                            store4<ODT, TO>(out + (int64_t)c_p * g.c_out + co0 + cl, v0, v1, v2, v3);
                    } else if constexpr (sizeof(TO) == 2) {
                        uint2 pk;
                        store4<ODT, TO>(reinterpret_cast<TO *>(&pk), v0, v1, v2, v3);
                        if (g.flags & FC_RELU) {
                            pk.x = relu_packed16(pk.x);
                            pk.y = relu_packed16(pk.y);
                        }
                        const uint32_t at = (uint32_t)l32 * 128u + (uint32_t)((b * 4 + q) ^ FC_SWZ(l32)) * 16u + (uint32_t)half * 8u;
                        *reinterpret_cast<uint2 *>(xs + at) = pk;
                    } else {
                        uint32_t pk;
                        store4<ODT, TO>(reinterpret_cast<TO *>(&pk), v0, v1, v2, v3);
                        if (g.flags & FC_RELU) pk = relu_packed8(pk);
                        const uint32_t at = (uint32_t)l32 * 128u + (uint32_t)((b * 2 + (q >> 1)) ^ FC_SWZ(l32)) * 16u +
                                            (uint32_t)((q & 1) * 8 + half * 4);
                        *reinterpret_cast<uint32_t *>(xs + at) = pk;
                    }
                }
            }
            if constexpr (sizeof(TO) <= 2) {
                __asm__ volatile("" ::: "memory");
                constexpr int EPT = 16 / (int)sizeof(TO);
                const bool inside = (lane & 7) * EPT < min(co_left, 64); // this lane's channels exist
                u32x4_t piece[4];
                int c_pr[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int row = j * 8 + (lane >> 3);
                    c_pr[j] = __shfl(c_p, row, 64);
                    piece[j] = *reinterpret_cast<const u32x4_t *>(xs + (uint32_t)row * 128u + (uint32_t)((lane & 7) ^ FC_SWZ(row)) * 16u);
                }
                // (the non-temporal stores are written out: the compiler folds a store and its non-temporal twin
                // into one plain store when they sit in the two arms of a branch)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    u32x4_t *at16 = reinterpret_cast<u32x4_t *>(out + (int64_t)(c_pr[j] < 0 ? 0 : c_pr[j]) * g.c_out + co0 + (lane & 7) * EPT);
                    if (c_pr[j] >= 0 && inside) {
                        if (stream_out)
                            __asm__ volatile("global_store_dwordx4 %0, %1, off nt" : : "v"(at16), "v"(piece[j]) : "memory");
                        else
                            *at16 = piece[j];
                    }
                }
                __asm__ volatile("" ::: "memory");
            }
        }
    }
}

// ---------------------------------------------------------------------------

// (shapes conv_pw_supported accepts, and unit horizontal stride and dilation)
bool conv_res3_supported(const Geom &g) { return g.kh == 3 && g.kw == 3 && g.sw == 1 && g.dw == 1; }

template <int DT, typename TO>
static hipError_t launch_res3(const Geom &g, int grid, bool bias_last, const void *x, const uint8_t *mask_in, const uint8_t *mask_out,
                              const void *w, const float *bias, const int32_t *idx, const int32_t *count, void *out, hipStream_t s)
{
    auto kern = k_conv_res3<DT, TO>;
    // the dynamic LDS limit is raised once per function and device
    static std::atomic<uint64_t> attr_devices{0};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t dev_bit = 1ull << (dev & 63);
    if (!(attr_devices.load(std::memory_order_acquire) & dev_bit)) {
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kResLdsBytes);
        if (e != hipSuccess) return e;
        attr_devices.fetch_or(dev_bit, std::memory_order_release);
    }
    const bool clears = mask_in && !(g.flags & (FC_SKIP_ZERO_FILL | FC_COMPACT_OUT));
    const int waves = kResWaves + (clears ? kResClearWaves : 0);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(waves * 64), kResLdsBytes, s, g, make_fastdiv((uint32_t)g.c_out * (uint32_t)sizeof(TO) / 16u), bias_last,
                       (const unsigned char *)x, mask_in, mask_out, (const unsigned char *)w, bias, idx, count, (TO *)out);
    return hipGetLastError();
}

hipError_t launch_conv_res3(const Geom &g, int in_dtype, int out_dtype, int grid, bool bias_last, const void *x, const uint8_t *mask_in,
                            const uint8_t *mask_out, const void *w, const float *bias, const int32_t *idx, const int32_t *count,
                            void *out, hipStream_t s)
{
#define FC_RES_CALL(DT, TO) launch_res3<DT, TO>(g, grid, bias_last, x, mask_in, mask_out, w, bias, idx, count, out, s)
    if (in_dtype == FC_BF16) {
        if (out_dtype == FC_F32) return FC_RES_CALL(FC_BF16, float);
        if (out_dtype == FC_FP8) return FC_RES_CALL(FC_BF16, uint8_t);
        return FC_RES_CALL(FC_BF16, uint16_t);
    }
    if (in_dtype == FC_FP8) {
        if (out_dtype == FC_F32) return FC_RES_CALL(FC_FP8, float);
        if (out_dtype == FC_FP8) return FC_RES_CALL(FC_FP8, uint8_t);
        return FC_RES_CALL(FC_FP8, uint16_t);
    }
    if (out_dtype == FC_F32) return FC_RES_CALL(FC_F16, float);
    if (out_dtype == FC_FP8) return FC_RES_CALL(FC_F16, uint8_t);
    return FC_RES_CALL(FC_F16, uint16_t);
#undef FC_RES_CALL
}

} // namespace fc
