// Focused convolution of fp32 storage (any channel counts from four on) and of grouped layers of 16-bit
// storage, on the matrix cores.
//
// Sec. III-A as everywhere: rows = kept positions, columns = output channels, reduction = taps
// x input channels, gated taps read as zero.  The two layer types share how rows are found and cleared; what
// bounds them differs:
//   - fp32: v_mfma_f32_32x32x2_f32 runs at 1/16 of the 16-bit rate, so large layers are bound by it; the operands
//     come through a ring of LDS stages, with a barrier per stage (k_conv_f32);
//   - grouped: a layer's multiplies are few (a ResNeXt stage: 0.24 GFLOP), its time is the
//     reading of x and the writing of out.  Weights stay in registers; the pixels come straight from global memory, a
//     tile or quad of rows ahead (k_conv_grouped, k_conv_grouped_quads), or, where positions are pixels, from one window
//     of pixels in LDS (k_conv_grouped_window).
//
// Rows.  A workgroup owns a span of consecutive positions.  Without a list it labels the span
// itself, compacts the kept positions in LDS and clears the rows of the others, so a masked call
// is one launch: no compaction before it, no zero-fill after it (they were 4 to 9 us and 4 to 5 us
// of launches around kernels that now take about as long).  With a list the span is a run of list
// entries, and the caller clears the irrelevant rows.
#include "fc_dma_util.hpp"
#include <type_traits>
#include <atomic>

namespace fc {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;

constexpr int kRegThreads = 256;
constexpr int kMaxSpan = 128;
constexpr int kGroupedSpan = 64;

// The rows of one workgroup's span, in LDS.
struct SpanRows {
    int32_t p[kMaxSpan];       // output position of row r
    int32_t base[kMaxSpan];    // input pixel under tap (0, 0) (may lie outside the image)
    int32_t hw[kMaxSpan];      // (ih, iw) of that pixel as two signed halves
    int32_t img[kMaxSpan];     // image number
    uint32_t bits[2][kMaxSpan];// tap t inside the image and relevant: bit t & 31 of word t >> 5
    int32_t dropped[kMaxSpan]; // irrelevant positions of the span
    int32_t waves[kMaxSpan / 64 + 1];
};

// Fills `s` for the span of S positions (or list entries) that starts at `first`; *nrows rows are
// to be computed, *ndrop to be cleared.  Called by all threads; ends with a barrier.
template <int S>
__device__ __forceinline__ void span_rows(const Geom &g, const uint8_t *__restrict__ mask_in,
                                          const uint8_t *__restrict__ mask_out, const int32_t *__restrict__ idx,
                                          int rows, int first, SpanRows &s, int *nrows, int *ndrop)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool packed = (g.flags & FC_PACKED_MASKS) != 0;
    int n = min(S, rows - first), nd = 0;
    if (mask_in && !idx) {
        const bool inside = tid < n;
        const bool kept = inside && position_kept(g, mask_in, mask_out, first + tid);
        const uint64_t k = __ballot(kept), d = __ballot(inside && !kept);
        if (S > 64 && lane == 0 && wave < S / 64) s.waves[wave] = __popcll(k);
        if (S > 64) __syncthreads();
        int kept_before = 0, total = 0;
        if (S > 64) {
#pragma unroll
            for (int v = 0; v < (S + 63) / 64; ++v) {
                kept_before += v < wave ? s.waves[v] : 0;
                total += s.waves[v];
            }
        } else {
            total = __popcll(k); // (only wave 0 holds positions; the others learn the total below)
        }
        const uint64_t below = (1ull << lane) - 1ull;
        if (kept) s.p[kept_before + __popcll(k & below)] = first + tid;
        if (inside && !kept) s.dropped[tid - lane - kept_before + __popcll(d & below)] = first + tid;
        if (S <= 64) {
            if (tid == 0) s.waves[0] = total;
            __syncthreads();
            total = s.waves[0];
        }
        nd = n - total;
        n = total;
    } else if (tid < n) {
        s.p[tid] = idx ? idx[first + tid] : first + tid;
    }
    __syncthreads();
    if (tid < S) {
        s.bits[0][tid] = 0u;
        s.bits[1][tid] = 0u;
        if (tid < n) {
            const int p = s.p[tid];
            const int q = (int)((uint32_t)p / (uint32_t)g.wo), ow = p - q * g.wo;
            const int b = (int)((uint32_t)q / (uint32_t)g.ho), oh = q - b * g.ho;
            const int ih = oh * g.sh - g.ph, iw = ow * g.sw - g.pw;
            s.base[tid] = (b * g.h + ih) * g.w + iw;
            s.hw[tid] = (int)(((uint32_t)ih & 0xffffu) | ((uint32_t)iw << 16));
            s.img[tid] = b;
        }
    }
    __syncthreads();
    // one thread per (row, tap): inside the image and relevant?
    const int taps = g.kh * g.kw;
    constexpr int U = 3; // look-ups of a thread in flight together
    for (int i0 = tid; i0 < n * taps; i0 += U * kRegThreads) {
        int row[U], tp[U], pix[U];
        uint32_t rel[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * kRegThreads;
            const bool some = i < n * taps;
            const int r = some ? (int)((uint32_t)i / (uint32_t)taps) : 0, t = some ? i - r * taps : 0;
            const int kh = (int)((uint32_t)t / (uint32_t)g.kw), kw = t - kh * g.kw;
            const int ih = (int)(int16_t)(s.hw[r] & 0xffff) + kh * g.dh, iw = (s.hw[r] >> 16) + kw * g.dw;
            const bool ok = some && ih >= 0 && ih < g.h && iw >= 0 && iw < g.w;
            row[u] = r;
            tp[u] = t;
            pix[u] = ok ? (s.img[r] * g.h + ih) * g.w + iw : -1;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) rel[u] = 1u;
        if (mask_in) {
#pragma unroll
            for (int u = 0; u < U; ++u) rel[u] = mask_at(mask_in, max(pix[u], 0), packed);
            loaded_together(rel);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (pix[u] >= 0 && rel[u]) atomicOr(&s.bits[tp[u] >> 5][row[u]], 1u << (tp[u] & 31));
    }
    __syncthreads();
    *nrows = n;
    *ndrop = nd;
}

// Clears channels [c0, c0 + nc) of the span's dropped rows; out_row = channels of a row.
template <typename TO>
__device__ __forceinline__ void clear_dropped(const SpanRows &s, int ndrop, TO *__restrict__ out, int out_row, int c0,
                                              int nc)
{
    constexpr int EPP = 16 / (int)sizeof(TO);
    if (out_row % EPP == 0 && c0 % EPP == 0 && nc % EPP == 0) {
        const int pieces = nc / EPP;
        const u32x4_t zero = {0u, 0u, 0u, 0u};
        for (int i = threadIdx.x; i < ndrop * pieces; i += kRegThreads) {
            const int r = (int)((uint32_t)i / (uint32_t)pieces), c = i - r * pieces;
            __builtin_nontemporal_store(zero, reinterpret_cast<u32x4_t *>(out + (int64_t)s.dropped[r] * out_row + c0 + c * EPP));
        }
    } else {
        for (int i = threadIdx.x; i < ndrop * nc; i += kRegThreads) {
            const int r = (int)((uint32_t)i / (uint32_t)nc), c = i - r * nc;
            out[(int64_t)s.dropped[r] * out_row + c0 + c] = TO(0);
        }
    }
}

// ---------------------------------------------------------------------------------------------
// fp32 storage.  Bound: the fp32 matrix rate (157 TFLOP/s) on large layers, the set-up's chain of
// dependent loads on small ones.
//
// One stage = 32 input channels (128 bytes) of one tap for the TM rows of the tile and its TN output
// channels, gathered straight into a ring of NB LDS buffers (swizzled as everywhere, see
// fc_dma_util.hpp).  Lane (row, half) of a wave reads the 16-byte piece 2 * kk + half of its row, and the
// four elements feed four v_mfma_f32_32x32x2_f32 whose reduction pair is (element e of the lower half,
// element e of the upper half); both operands are read the same way, so the pairing of
// channels is the same.  (Operands loaded from global memory straight into registers need no
// barrier but put every lane of a load on another line: 64 cycles of address work each, and the large
// layers stop at 77 TFLOP/s.)
//
// WK = 4: the four waves take the same 32 rows and every fourth kk of each stage, two stages
// between barriers, and add up through LDS in wave order: a layer of a few hundred row blocks is spread
// over four times as many SIMDs.  WK = 1: 32 rows of a 128-position span each.
// TAIL: the input channels are not whole 32-channel stages.
//
// Measured (mask given, call and output tensor included): 64 -> 64 on 2 x 60 x 80, half kept: 75.8 us on the vector
// ALUs with a compaction and a zero-fill launch, 15.9 us; 128 -> 128 on 8 x 120 x 120 without a mask: 321 us =
// 106 TFLOP/s.
// ---------------------------------------------------------------------------------------------
template <int TN, int WK, int NB, bool TAIL>
__global__ __launch_bounds__(kRegThreads, 2) void k_conv_f32(Geom g, const float *__restrict__ x,
                                                             const uint8_t *__restrict__ mask_in,
                                                             const uint8_t *__restrict__ mask_out,
                                                             const float *__restrict__ w,
                                                             const float *__restrict__ bias,
                                                             const int32_t *__restrict__ idx,
                                                             const int32_t *__restrict__ count, float *__restrict__ out)
{
    constexpr int TM = WK == 4 ? 32 : 128;
    constexpr int CB = TN / 32;              // 32-channel blocks of a wave
    constexpr int XR = TM / 32, WR = TN / 32;// loads per thread and stage
    constexpr int L = XR + WR;
    constexpr int R = WK == 4 ? 2 : 1;       // stages between two barriers
    constexpr uint32_t STAGE = (uint32_t)(TM + TN) * 128u;
    static_assert(NB % R == 0 && NB >= 2 * R && NB * L <= 63, "vmcnt is a 6-bit counter");
    static_assert(WK == 1 || NB * STAGE >= 4u * CB * 4u * 64u * 16u, "the partial sums fit the stage buffers");
    __shared__ __align__(16) unsigned char stage[NB * STAGE];
    __shared__ SpanRows rows_s;
    const int rows = idx ? *count : g.m;
    const int first = blockIdx.x * TM;
    if (first >= rows) return;
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int co0 = blockIdx.y * TN;
    int n, nd;
    span_rows<TM>(g, mask_in, mask_out, idx, rows, first, rows_s, &n, &nd);
    if (nd && !(g.flags & FC_SKIP_ZERO_FILL)) clear_dropped<float>(rows_s, nd, out, g.c_out, co0, min(TN, g.c_out - co0));
    if (n == 0) return;

    const int taps = g.kh * g.kw;
    // a row's offset is that of its first tap, which may lie in front of the tensor: x is read through a
    // descriptor that starts a padding's worth earlier (those taps are switched off, nothing in front
    // of the tensor is read), so that the per-lane part of an offset is never negative
    // (TAIL: x and w through descriptors that start one piece earlier still, since a row's last piece may begin before the lane's own offset, 33
    // channels at three of the first chunk's, and the range is checked before a stage's scalar offset is added)
    constexpr uint32_t lead = TAIL ? 16u : 0u;
    const uint32_t xbias = (uint32_t)(g.ph * g.w + g.pw) * (uint32_t)g.c_in * 4u + lead;
    const u32x4_t rsrc_x = make_rsrc_words(reinterpret_cast<const unsigned char *>(x) - xbias,
                                           (uint32_t)g.n * g.h * g.w * g.c_in * 4u + xbias);
    const u32x4_t rsrc_w = make_rsrc_words(reinterpret_cast<const unsigned char *>(w) - lead, (uint32_t)g.c_out * taps * g.c_in * 4u + lead);
    // A row whose length is no multiple of four ends in a piece of its last four channels, of which the
    // first `again` were already in the piece before it: they are cleared in both operands.  `edge` = first
    // channel of that piece.
    const int again = TAIL ? (4 - (g.c_in & 3)) & 3 : 0, edge = again ? g.c_in - 4 + again : -1;
    const int cch = (g.c_in + 31) >> 5, stages = taps * cch;
    const int last_steps = (g.c_in - (cch - 1) * 32 + 7) >> 3; // 8-channel steps of a tap's last stage
    const int slot = tid & 7, prow = tid >> 3;
    const int piece = slot ^ FC_SWZ(prow); // (the rows of a thread's loads differ by multiples of 32)
    uint32_t xoff[XR], woff[WR];
    uint32_t xbits[2][XR];
#pragma unroll
    for (int j = 0; j < XR; ++j) {
        const int r = prow + j * 32;
        const bool live = r < n;
        xoff[j] = live ? (uint32_t)(rows_s.base[r] * g.c_in + piece * 4) * 4u + xbias : 0u;
        xbits[0][j] = live ? rows_s.bits[0][r] : 0u;
        xbits[1][j] = live ? rows_s.bits[1][r] : 0u;
    }
#pragma unroll
    for (int j = 0; j < WR; ++j) {
        const int co = co0 + prow + j * 32;
        woff[j] = co < g.c_out ? (uint32_t)(co * taps * g.c_in + piece * 4) * 4u + lead : kOutOfRange;
    }
    const uint32_t lds0 =
        __builtin_amdgcn_readfirstlane((uint32_t)reinterpret_cast<uintptr_t>(stage) + (uint32_t)wave * 1024u);

    // cursor of the next stage to load (stages past the end load zeros)
    int tap = 0, cc = 0, kh = 0, kw = 0, ibuf = 0;
    auto issue = [&]() __attribute__((always_inline)) {
        const bool in_k = tap < taps;
        uint32_t sx = in_k ? (uint32_t)((kh * g.dh * g.w + kw * g.dw) * g.c_in + cc * 32) * 4u : 0u;
        uint32_t sw = in_k ? (uint32_t)(tap * g.c_in + cc * 32) * 4u : 0u;
        sx = __builtin_amdgcn_readfirstlane(sx);
        sw = __builtin_amdgcn_readfirstlane(sw);
        __asm__("" : "+s"(sx), "+s"(sw)); // (registers, not constants: the load takes no literal there)
        const uint32_t sel = in_k ? 1u << (tap & 31) : 0u;
        const int ch = cc * 32 + piece * 4;
        const bool in = !TAIL || ch < g.c_in;
        const uint32_t back = TAIL && ch == edge ? (uint32_t)again * 4u : 0u;
        const uint32_t to = lds0 + (uint32_t)ibuf * STAGE;
#pragma unroll
        for (int j = 0; j < XR; ++j) {
            const bool ok = ((tap < 32 ? xbits[0][j] : xbits[1][j]) & sel) && in;
            dma_load16_s(rsrc_x, ok ? xoff[j] - back : kOutOfRange, sx, to + (uint32_t)j * 4096u);
        }
#pragma unroll
        for (int j = 0; j < WR; ++j)
            dma_load16_s(rsrc_w, in_k && in && woff[j] != kOutOfRange ? woff[j] - back : kOutOfRange, sw,
                         to + (uint32_t)(XR + j) * 4096u);
        ibuf = ibuf + 1 == NB ? 0 : ibuf + 1;
        if (++cc == cch) {
            cc = 0;
            ++tap;
            if (++kw == g.kw) {
                kw = 0;
                ++kh;
            }
        }
    };

    f32x16_t acc[CB];
#pragma unroll
    for (int b = 0; b < CB; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[b][i] = 0.f;
#pragma unroll
    for (int d = 0; d < NB - R; ++d) issue();

    const uint32_t frag = (uint32_t)l32 * 128u;
    const int wm = WK == 4 ? 0 : wave;
    int mcc = 0, cbuf = 0; // channel chunk and buffer of the stage to multiply
    // (an odd number of stages: the last round's second stage is one past the end, all zeros)
    for (int s = 0; s < stages; s += R) {
        wait_vmcnt<(NB - 2 * R) * L>(); // this thread's loads of the round's stages have landed
        __syncthreads();                // ... and everyone else's; the buffers of the round before are free
#pragma unroll
        for (int d = 0; d < R; ++d) issue();
#pragma unroll
        for (int d = 0; d < R; ++d) {
            const unsigned char *xs = stage + (uint32_t)cbuf * STAGE + (uint32_t)wm * 4096u + frag;
            const unsigned char *ws = stage + (uint32_t)cbuf * STAGE + (uint32_t)TM * 128u + frag;
            const bool last = mcc + 1 == cch;
            const int steps = TAIL && last ? last_steps : 4;
#pragma unroll
            for (int kq = 0; kq < 4 / WK; ++kq) {
                const int kk = WK == 4 ? wave : kq;
                if (TAIL && kk >= steps) break;
                const uint32_t o = (uint32_t)((2 * kk + half) ^ FC_SWZ(l32)) * 16u;
                float4 xv = *reinterpret_cast<const float4 *>(xs + o), wv[CB];
#pragma unroll
                for (int b = 0; b < CB; ++b) wv[b] = *reinterpret_cast<const float4 *>(ws + b * 4096 + o);
                if (TAIL && last && again && kk == steps - 1) {
                    const int drop = mcc * 32 + (2 * kk + half) * 4 == edge ? again : 0;
                    xv.x = drop > 0 ? 0.f : xv.x;
                    xv.y = drop > 1 ? 0.f : xv.y;
                    xv.z = drop > 2 ? 0.f : xv.z;
#pragma unroll
                    for (int b = 0; b < CB; ++b) {
                        wv[b].x = drop > 0 ? 0.f : wv[b].x;
                        wv[b].y = drop > 1 ? 0.f : wv[b].y;
                        wv[b].z = drop > 2 ? 0.f : wv[b].z;
                    }
                }
                const float xe[4] = {xv.x, xv.y, xv.z, xv.w};
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int b = 0; b < CB; ++b) {
                        const float we = e == 0 ? wv[b].x : e == 1 ? wv[b].y : e == 2 ? wv[b].z : wv[b].w;
                        acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(we, xe[e], acc[b], 0, 0, 0);
                    }
            }
            mcc = last ? 0 : mcc + 1;
            cbuf = cbuf + 1 == NB ? 0 : cbuf + 1;
        }
    }
    wait_vmcnt<0>();

    // a lane's quad (b, q) = channels co0 + 32 b + 8 q + 4 half .. + 3 of the position of row r; the bias of all its quads comes in one
    // round trip (where it was used, each value had one of its own: 128 -> 128 without a mask on 8 x 120 x 120 323 -> 315 us, half kept 246 -> 239)
    constexpr int NQ = WK == 4 ? 1 : 4; // quads of a block that a lane finishes
    float bq[CB * NQ * 4];
    if (bias) {
#pragma unroll
        for (int b = 0; b < CB; ++b)
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    bq[(b * NQ + q) * 4 + i] = bias[min(co0 + b * 32 + (WK == 4 ? wave : q) * 8 + half * 4 + i, g.c_out - 1)];
        loaded_together(bq);
    }
    const int r = wm * 32 + l32;
    const int64_t at = r < n ? (int64_t)rows_s.p[r] * g.c_out : -1;
    auto finish = [&](int b, int q, float4 v) __attribute__((always_inline)) {
        const int co = co0 + b * 32 + q * 8 + half * 4;
        float e[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (bias) e[i] += bq[(b * NQ + (WK == 4 ? 0 : q)) * 4 + i];
            if (g.flags & FC_RELU) e[i] = !(e[i] > 0.f) ? (e[i] != e[i] ? e[i] : 0.f) : e[i];
        }
        if (at < 0) return;
        if ((g.c_out & 3) == 0) {
            if (co < g.c_out) *reinterpret_cast<float4 *>(out + at + co) = make_float4(e[0], e[1], e[2], e[3]);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (co + i < g.c_out) out[at + co + i] = e[i];
        }
    };
    if constexpr (WK == 4) {
        __syncthreads(); // every wave is done with the stage buffers
        float4 *part = reinterpret_cast<float4 *>(stage);
#pragma unroll
        for (int b = 0; b < CB; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                part[((wave * CB + b) * 4 + q) * 64 + lane] =
                    make_float4(acc[b][q * 4], acc[b][q * 4 + 1], acc[b][q * 4 + 2], acc[b][q * 4 + 3]);
        __syncthreads();
        // wave v finishes quad v of every 32-channel block
#pragma unroll
        for (int b = 0; b < CB; ++b) {
            float4 v = part[(b * 4 + wave) * 64 + lane];
#pragma unroll
            for (int k = 1; k < 4; ++k) {
                const float4 t = part[((k * CB + b) * 4 + wave) * 64 + lane];
                v.x += t.x; v.y += t.y; v.z += t.z; v.w += t.w;
            }
            finish(b, wave, v);
        }
    } else {
#pragma unroll
        for (int b = 0; b < CB; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                finish(b, q, make_float4(acc[b][q * 4], acc[b][q * 4 + 1], acc[b][q * 4 + 2], acc[b][q * 4 + 3]));
    }
}

// ---------------------------------------------------------------------------------------------
// The same split (WK = 4) for 3x3 kernels, horizontally undilated, with bytes for masks: what bounds k_conv_f32 there is not
// the matrix cores (two workgroups of a CU: 9 200 cycles) but what its waves issue beside them: stamps of 64 -> 64 on 2 x 60 x 80, half
// kept, 5 100 cycles to the rows' bits (three divisions by run-time numbers a look-up, five barriers), 13 500 in the stages, 3 500 from there to
// the last store.  Here
//   - a lane holds a row: consecutive positions (rows are 32 a tile, so compacting them saves no instruction), or list entries; every
//     wave finds all 32 by itself, no barrier;
//   - what the mask says about a row's taps selects the LDS address its operand is read from: the row's, or one of zeros;
//   - lane q knows the offsets of stage q; a load is an addition and an instruction;
//   - a round is three stages with one barrier, two rounds are on their way, LDS offsets are constants.
// The products, their order and the order of the four waves' sums are those of k_conv_f32.  Mask given, one launch after
// another, half kept, us: 64 -> 64 on 2 x 60 x 80 15.5 -> 10.4, 32 -> 32 on 14 x 20 7.3 -> 4.6, 64 -> 66 on 8 x 30 x 40 stride 2 9.7 -> 6.6, 96 -> 128 on 4 x 67 x 90
// 60.5 -> 46.6.
// ---------------------------------------------------------------------------------------------
constexpr int kF32Round = 3;
constexpr uint32_t kF32Stage = 64u * 128u;
template <int RING> constexpr uint32_t kF32Zeros = RING * kF32Round * kF32Stage;
template <int RING> constexpr uint32_t kF32Lds = kF32Zeros<RING> + 128u;
constexpr int kF32MostStages = 63; // a lane each

// RING: rounds in LDS; TAIL: the input channels are not whole 32-channel stages
template <int RING, bool TAIL>
__global__ __launch_bounds__(kRegThreads, RING == 2 ? 3 : 2) void k_conv_f32_rounds(Geom g, FastDiv by_cch, const float *__restrict__ x,
                                                                    const uint8_t *__restrict__ mask_in,
                                                                    const uint8_t *__restrict__ mask_out,
                                                                    const float *__restrict__ w,
                                                                    const float *__restrict__ bias,
                                                                    const int32_t *__restrict__ idx,
                                                                    const int32_t *__restrict__ count, float *__restrict__ out)
{
    extern __shared__ __align__(16) unsigned char lds[];
    const int rows = idx ? __builtin_amdgcn_readfirstlane(*count) : g.m;
    const int first = blockIdx.x * 32;
    if (first >= rows) return;
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int co0 = blockIdx.y * 32;

    // ---- request what decides about the rows ----
    int p = first + l32;
    bool live = p < rows;
    // (values of loads that are waited for by hand are touched by nothing before the wait; by a scalar, so that no path leads from one load to the other)
    const int by_list = TAIL ? __builtin_amdgcn_readfirstlane(idx != nullptr ? 1 : 0) : idx != nullptr;
    uint32_t entry, label;
    if (by_list) {
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
    const int co = co0 + wave * 8 + half * 4;

    // ---- stages: wave v loads rows 8 v .. 8 v + 7 of the pixels and of the weights ----
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)reinterpret_cast<uintptr_t>(lds) + (uint32_t)wave * 1024u);
    const int prow = wave * 8 + (lane >> 3);
    const uint32_t piece = (uint32_t)((lane & 7) ^ FC_SWZ(prow)) * 16u;
    const uint32_t pixel = (uint32_t)g.c_in * 4u, wrow = 9u * pixel;
    const int cch = TAIL ? (g.c_in + 31) >> 5 : g.c_in >> 5, stages = 9 * cch;
    const u32x4_t rsrc_w = make_rsrc_words(w, (uint32_t)g.c_out * wrow);
    uint32_t woff = (uint32_t)(co0 + prow) * wrow + piece;
    __asm__("" : "+v"(woff));
    woff = co0 + prow < g.c_out ? woff : kOutOfRange;
    const int tap_q = (int)fast_div((uint32_t)lane, by_cch), kh_q = tap_q * 11 >> 5, cc_q = lane - tap_q * cch;
    // (TAIL: bit 31 marks the last stage of a tap)
    const int bit_q = TAIL ? 1 << (tap_q & 15) | (cc_q + 1 == cch ? 1 << 31 : 0) : 1 << (tap_q & 31);
    const int x_q = (kh_q * g.dh * g.w + (tap_q - 3 * kh_q)) * (int)pixel + cc_q * 128, w_q = tap_q * (int)pixel + cc_q * 128;
    // TAIL: what a tap's last stage loads: nothing past the last channel, and a row whose length is no multiple of four ends in a piece of
    // its last four channels, of which the first `again` were already in the piece before it: they are cleared in both operands.
    const uint32_t left = (uint32_t)(g.c_in - (cch - 1) * 32) * 4u; // bytes of that stage
    const int again = TAIL ? (4 - (g.c_in & 3)) & 3 : 0;
    const uint32_t back = again && piece == (left & ~15u) ? (uint32_t)again * 4u : 0u;
    const bool past = piece >= left;
    const uint32_t woff_last = past || woff == kOutOfRange ? kOutOfRange : woff - back;
    const int cleared = 2 * wave + half == (int)(left >> 4) ? again : 0; // of the piece that this lane multiplies
    if (tid < 8) *reinterpret_cast<uint4 *>(lds + kF32Zeros<RING> + tid * 16) = make_uint4(0u, 0u, 0u, 0u);

    // ---- the rows ----
    wait_vmcnt<0>();
    bool drop = false;
    if (by_list) {
        __asm__ volatile("" : "+v"(entry)::"memory");
        p = live ? (int)entry : 0;
    } else if (mask_in) {
        __asm__ volatile("" : "+v"(label)::"memory");
        const bool kept = live && label != 0;
        drop = live && !kept;
        live = kept;
    }
    const bool fill = mask_in && !idx && !(g.flags & FC_SKIP_ZERO_FILL);
    float *const to = out + (int64_t)(drop ? first + l32 : p) * g.c_out + co;
    auto store = [&](float4 v) __attribute__((always_inline)) {
        if (!(live || (drop && fill))) return;
        const float e[4] = {drop ? 0.f : v.x, drop ? 0.f : v.y, drop ? 0.f : v.z, drop ? 0.f : v.w};
        if ((g.c_out & 3) == 0) {
            if (co < g.c_out) *reinterpret_cast<float4 *>(to) = make_float4(e[0], e[1], e[2], e[3]);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (co + i < g.c_out) to[i] = e[i];
        }
    };
    if (__ballot(live) == 0) { // (the same in all waves; nothing is on its way to a register here)
        store(make_float4(0.f, 0.f, 0.f, 0.f));
        return;
    }
    const int pp = live ? p : 0;
    const int q = (int)fast_div((uint32_t)pp, g.div_wo), ow = pp - q * g.wo;
    const int img = (int)fast_div((uint32_t)q, g.div_ho), oh = q - img * g.ho;
    const int ih0 = oh * g.sh - g.ph, iw0 = ow * g.sw - g.pw;
    const int pix0 = (img * g.h + ih0) * g.w + iw0; // may lie outside the image

    // the bias of the channels this lane stores, added at the end
    const u32x4_t rsrc_b = make_rsrc_words(bias, bias ? (uint32_t)g.c_out * 4u : 0u);
    uint32_t bq[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        __asm__ volatile("buffer_load_dword %0, %1, %2, 0 offen" : "=v"(bq[i]) : "v"((uint32_t)(co + i) * 4u), "s"(rsrc_b) : "memory");
    // the mask bytes under the taps of a kernel row with one (unaligned) 4-byte load each; one that would leave the
    // mask is moved inside it and its bytes moved back (without a mask: three loads of something, not looked at)
    const uint8_t *const from = mask_in ? mask_in : reinterpret_cast<const uint8_t *>(w);
    const int most = mask_in ? g.n * g.h * g.w - 4 : 0;
    uint32_t m[3];
    int moved[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int off = pix0 + k * g.dh * g.w, at = min(max(off, 0), most);
        moved[k] = off - at;
        __asm__ volatile("global_load_dword %0, %1, %2" : "=v"(m[k]) : "v"(at), "s"(from) : "memory");
    }
    const u32x4_t rsrc_x = make_rsrc_words(x, (uint32_t)g.n * g.h * g.w * pixel);
    // (what lies outside the tensor is out of range, whichever side; what lies in it beside the image is not looked at)
    const uint32_t xoff = (uint32_t)__shfl(pix0, prow) * pixel + piece;
    const uint32_t xoff_last = past ? kOutOfRange : xoff - back; // (out of range with a tap's offset added, see f32_rounds)
    auto load_round = [&](int s, int slot) __attribute__((always_inline)) {
        uint32_t sx[kF32Round], sw[kF32Round];
#pragma unroll
        for (int d = 0; d < kF32Round; ++d) {
            sx[d] = (uint32_t)__builtin_amdgcn_readlane(x_q, s + d);
            sw[d] = (uint32_t)(s + d) * 128u;
            __asm__ volatile("" : "+s"(sw[d]));
        }
        if constexpr (TAIL) {
            uint32_t ox[kF32Round], ow[kF32Round];
#pragma unroll
            for (int d = 0; d < kF32Round; ++d) {
                const bool last = __builtin_amdgcn_readlane(bit_q, s + d) < 0;
                ox[d] = (last ? xoff_last : xoff) + sx[d];
                // (by the vector unit: what it wrote into a scalar register may not be a load's scalar offset right after)
                ow[d] = (last ? woff_last : woff) + (uint32_t)__builtin_amdgcn_readlane(w_q, s + d);
            }
#pragma unroll
            for (int d = 0; d < kF32Round; ++d) {
                dma_load16(rsrc_x, ox[d], lds0 + (uint32_t)(slot + d) * kF32Stage);
                dma_load16(rsrc_w, ow[d], lds0 + (uint32_t)(slot + d) * kF32Stage + 4096u);
            }
            return;
        }
#pragma unroll
        for (int d = 0; d < kF32Round; ++d) {
            dma_load16(rsrc_x, xoff + sx[d], lds0 + (uint32_t)(slot + d) * kF32Stage);
            dma_load16_s(rsrc_w, woff, sw[d], lds0 + (uint32_t)(slot + d) * kF32Stage + 4096u);
        }
    };
#pragma unroll
    for (int r = 0; r < RING - 1; ++r) load_round(r * kF32Round, r * kF32Round);

    // taps inside the image and relevant
    uint32_t bits = 0, rel = 0, cols = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k) cols |= (uint32_t)(iw0 + k) < (uint32_t)g.w ? 1u << k : 0u;
#pragma unroll
    for (int k = 0; k < 3; ++k) bits |= (uint32_t)(ih0 + k * g.dh) < (uint32_t)g.h ? cols << (3 * k) : 0u;
    wait_vmcnt<(RING - 1) * 2 * kF32Round>();
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        __asm__ volatile("" : "+v"(m[k])::"memory");
        uint32_t v = moved[k] < 0 ? (moved[k] > -4 ? m[k] << (-8 * moved[k]) : 0u) : (moved[k] < 4 ? m[k] >> (8 * moved[k]) : 0u);
        v = (((v & 0x7f7f7f7fu) + 0x7f7f7f7fu) | v) & 0x80808080u; // nonzero bytes
        rel |= (((v >> 7) & 1u) | ((v >> 14) & 2u) | ((v >> 21) & 4u)) << (3 * k);
    }
    bits = live ? bits & (mask_in ? rel : ~0u) : 0u;

    f32x16_t acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
    const uint32_t at = (uint32_t)l32 * 128u + (uint32_t)((2 * wave + half) ^ FC_SWZ(l32)) * 16u;
    auto round = [&](int s, int r) __attribute__((always_inline)) {
        if (RING == 2 || s + kF32Round == stages) wait_vmcnt<0>();
        else wait_vmcnt<(RING - 2) * 2 * kF32Round>(); // this round's stages have landed
        __syncthreads();                               // ... all waves' parts; the round before is read
        float4 xv[kF32Round], wv[kF32Round];
#pragma unroll
        for (int d = 0; d < kF32Round; ++d) {
            const uint32_t slot = (uint32_t)(r * kF32Round + d) * kF32Stage;
            const bool on = bits & (uint32_t)__builtin_amdgcn_readlane(bit_q, s + d);
            xv[d] = *reinterpret_cast<const float4 *>(lds + slot + (on ? at : kF32Zeros<RING> - slot));
            wv[d] = *reinterpret_cast<const float4 *>(lds + slot + 4096u + at);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (TAIL && again) // uniform
#pragma unroll
            for (int d = 0; d < kF32Round; ++d) {
                const int drop = __builtin_amdgcn_readlane(bit_q, s + d) < 0 ? cleared : 0;
                xv[d].x = drop > 0 ? 0.f : xv[d].x; wv[d].x = drop > 0 ? 0.f : wv[d].x;
                xv[d].y = drop > 1 ? 0.f : xv[d].y; wv[d].y = drop > 1 ? 0.f : wv[d].y;
                xv[d].z = drop > 2 ? 0.f : xv[d].z; wv[d].z = drop > 2 ? 0.f : wv[d].z;
            }
        if (s + (RING - 1) * kF32Round < stages) load_round(s + (RING - 1) * kF32Round, (r + RING - 1) % RING * kF32Round);
#pragma unroll
        for (int d = 0; d < kF32Round; ++d) {
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wv[d].x, xv[d].x, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wv[d].y, xv[d].y, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wv[d].z, xv[d].z, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wv[d].w, xv[d].w, acc, 0, 0, 0);
        }
    };
    for (int s = 0; s < stages; s += RING * kF32Round) {
#pragma unroll
        for (int r = 0; r < RING; ++r)
            if (RING == 3 || r == 0 || s + r * kF32Round < stages) round(s + r * kF32Round, r); // (the rounds are a multiple of three)
    }
    // wave v finishes quad v: channels co0 + 8 v + 4 half .. + 3 of the position of row l & 31
    __syncthreads(); // every wave is done with the stages
    float4 *part = reinterpret_cast<float4 *>(lds);
#pragma unroll
    for (int k = 0; k < 4; ++k) part[(wave * 4 + k) * 64 + lane] = make_float4(acc[k * 4], acc[k * 4 + 1], acc[k * 4 + 2], acc[k * 4 + 3]);
    __syncthreads();
    float4 v = part[wave * 64 + lane];
#pragma unroll
    for (int k = 1; k < 4; ++k) {
        const float4 t = part[(k * 4 + wave) * 64 + lane];
        v.x += t.x; v.y += t.y; v.z += t.z; v.w += t.w;
    }
    float e[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        __asm__ volatile("" : "+v"(bq[i])::"memory");
        if (bias) e[i] += __uint_as_float(bq[i]);
        if (g.flags & FC_RELU) e[i] = !(e[i] > 0.f) ? (e[i] != e[i] ? e[i] : 0.f) : e[i];
    }
    store(make_float4(e[0], e[1], e[2], e[3]));
}

static bool f32_rounds(const Geom &g, bool masked)
{
    // (channels past whole chunks: a piece past the last one stays out of range with the offset of any stage added, two rows and two pixels
    // and less than a pixel more)
    return g.kh == 3 && g.kw == 3 && g.dw == 1 && 9 * ((g.c_in + 31) / 32) <= kF32MostStages &&
           (g.c_in % 32 == 0 || ((int64_t)g.dh * g.w * 2 + 3) * g.c_in * 4 < (int64_t)(0xffffffffu - kOutOfRange)) &&
           (!masked || (!(g.flags & FC_PACKED_MASKS) && (int64_t)g.n * g.h * g.w >= 4));
}

template <int RING, bool TAIL>
static hipError_t launch_f32_ring(const Geom &g, const void *x, const uint8_t *mask_in, const uint8_t *mask_out, const void *w,
                                    const float *bias, const int32_t *idx, const int32_t *count, void *out, hipStream_t s)
{
    // (more than 64 KB of dynamic LDS: allowed once per device)
    static std::atomic<uint64_t> attr_devices{0};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t dev_bit = 1ull << (dev & 63);
    if (!(attr_devices.load(std::memory_order_acquire) & dev_bit)) {
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_conv_f32_rounds<RING, TAIL>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kF32Lds<RING>);
        if (e != hipSuccess) return e;
        attr_devices.fetch_or(dev_bit, std::memory_order_release);
    }
    hipLaunchKernelGGL((k_conv_f32_rounds<RING, TAIL>), dim3((g.m + 31) / 32, (g.c_out + 31) / 32), dim3(kRegThreads), kF32Lds<RING>, s, g,
                       make_fastdiv((uint32_t)((g.c_in + 31) / 32)), (const float *)x, mask_in, mask_out, (const float *)w, bias, idx, count, (float *)out);
    return hipGetLastError();
}

static hipError_t launch_f32_rounds(const Geom &g, const void *x, const uint8_t *mask_in, const uint8_t *mask_out, const void *w,
                                    const float *bias, const int32_t *idx, const int32_t *count, void *out, hipStream_t s)
{
    // Three workgroups of a CU with two rounds each, or two with three.  Three hide each other's waits better (128 -> 128 without a mask on 3 x 50 x 50
    // 29.2 -> 28.6 us), but where there is work for two a CU some CUs get three and others one.  Of the tiles of a mask of regions about 17 in 20
    // hold a kept row; a list's rows fill no more than they have to.  Mask alone, 0.3 / 0.5 / 0.7 kept, two rounds -> three: 64 -> 64 on
    // 2 x 60 x 80 (600 tiles) 11.7 / 12.9 / 13.3 -> 10.8 / 11.2 / 11.6, 192 -> 128 on 56 x 80 (560) 25.5 / 25.8 / 28.3 -> 21.8 / 22.3 / 22.6, 64 -> 64 on 2 x 55 x 88 (606) 11.7 / 13.0 /
    // 13.3 -> 10.8 / 11.5 / 15.0, on 100 x 98 (614) 11.5 / 11.9 / 12.9 -> 10.7 / 12.2 / 14.9, 96 -> 128 on 2 x 50 x 50 (628) 16.9 / 17.4 / 17.7 -> 15.8 / 19.8 / 20.4; few tiles, 64 -> 64 on 60 x 80
    // (300) 9.5 / 9.6 / 9.7 -> 9.3 / 9.4 / 9.4.  With a list 2 x 60 x 80 12.9 / 13.6 / 14.3 -> 12.7 / 13.4 / 14.3, 128 -> 128 on 72 x 75 (676) 20.6 / 21.5 / 26.4 -> 20.8 / 21.5 /
    // 21.8, on 3 x 50 x 50 (940) 26.3 / 27.0 / 28.0 -> 21.6 / 22.7 / 33.3.  Masks that keep nine tenths fill more tiles than that: 2 x 60 x 80 13.6 -> 16.8, with a list 17.1 -> 19.6.
    const int64_t tiles = (int64_t)((g.m + 31) / 32) * ((g.c_out + 31) / 32), busy = idx ? tiles * 7 / 10 : mask_in ? tiles * 17 / 20 : tiles;
    const int cus = conv_grid_cus();
#define FC_RING(RING)                                                                                                        \
    (g.c_in % 32 ? launch_f32_ring<RING, true>(g, x, mask_in, mask_out, w, bias, idx, count, out, s)                         \
                 : launch_f32_ring<RING, false>(g, x, mask_in, mask_out, w, bias, idx, count, out, s))
    return busy > cus && busy <= 2 * cus ? FC_RING(3) : FC_RING(2);
#undef FC_RING
}

// four channels: one piece; 64 taps: the tap-valid bits of a row; 32-bit byte offsets into x and w; row
// origins in 16 bits
bool conv_f32_supported(const Geom &g)
{
    return g.c_in >= 4 && g.kh * g.kw <= 64 && g.h <= 16384 && g.w <= 16384 && g.ph <= 8192 && g.pw <= 8192 &&
           ((uint64_t)g.n * g.h * g.w + (uint64_t)g.ph * g.w + g.pw) * g.c_in * 4u + 16u < kBufferLimit &&
           (uint64_t)g.c_out * g.kh * g.kw * g.c_in * 4u + 16u < kBufferLimit; // (16: the piece a descriptor may start earlier)
}

template <int TN, int WK, int NB, bool TAIL>
static hipError_t launch_f32(const Geom &g, const void *x, const uint8_t *mask_in, const uint8_t *mask_out, const void *w,
                             const float *bias, const int32_t *idx, const int32_t *count, void *out, hipStream_t s)
{
    constexpr int TM = WK == 4 ? 32 : 128;
    hipLaunchKernelGGL((k_conv_f32<TN, WK, NB, TAIL>), dim3((g.m + TM - 1) / TM, (g.c_out + TN - 1) / TN), dim3(kRegThreads), 0,
                       s, g, (const float *)x, mask_in, mask_out, (const float *)w, bias, idx, count, (float *)out);
    return hipGetLastError();
}

hipError_t launch_conv_f32(const Geom &g, const void *x, const uint8_t *mask_in, const uint8_t *mask_out, const void *w,
                           const float *bias, const int32_t *idx, const int32_t *count, void *out, hipStream_t s)
{
    // 64 output channels per tile halve the gathering of x; an odd number of 32-channel blocks would
    // leave half of the last tile idle
    const int blocks32 = (g.c_out + 31) / 32;
    const bool wide = blocks32 % 2 == 0;
#define FC_F32(TN, WK, NB)                                                                                     \
    (g.c_in % 32 ? launch_f32<TN, WK, NB, true>(g, x, mask_in, mask_out, w, bias, idx, count, out, s)          \
                 : launch_f32<TN, WK, NB, false>(g, x, mask_in, mask_out, w, bias, idx, count, out, s))
    // Split the reduction when a wave per 32 rows would give fewer than one wave per SIMD, or, with a mask,
    // four: spans without a kept row leave their CUs to the others, which the smaller spans even out
    // (95 -> 116 on 4 x 67 x 90, half of it kept: 73 -> 67 us; without a mask 33 -> 65 on 4 x 90 x 90 loses,
    // 47 -> 53 us).  32 output channels then: 64 halve the workgroups (64 -> 64 on 2 x 60 x 80: 15.6 and 17.5 us).
    const int64_t waves = (int64_t)((g.m + 31) / 32) * (wide ? blocks32 / 2 : blocks32);
    // (k_conv_f32_rounds without a mask too: 96 -> 128 on 4 x 67 x 90 70 -> 58 us, 128 -> 64 on 3 x 100 x 110 88 -> 56; 128 -> 128 on 8 x 120 x 120, 7 200
    // waves, 322 -> 332, with a mask 233 / 244 / 251 -> 175 / 229 / 267 at 0.3 / 0.5 / 0.7 kept)
    // Channels past whole chunks are a quarter to three quarters of a stage that its four waves wait for together.  Mask given, us, general
    // kernel -> rounds: 76 -> 40 on 4 x 91 x 51 30.2 -> 22.7, 16 -> 56 on 7 x 32 x 89 19.7 -> 13.9, 21 -> 44 on 2 x 17 x 38 8.6 -> 5.7, 100 -> 110 on
    // 5 x 54 x 102 91.6 -> 75.7, 20 -> 128 on 8 x 120 x 120 66.8 -> 67.0.  Without a mask as much while a wave a block of rows is too few (52 -> 73 on 2 x
    // 57 x 26 12.7 -> 10.1); then that wave, which multiplies no padding, is better unless there is next to none: 100 -> 110 on 5 x 54 x 102 (13 of 16
    // steps) 81 -> 91, 33 -> 65 on 4 x 90 x 90 (5 of 8) 42 -> 49, but 95 -> 116 on 4 x 67 x 90 (12 of 12) 71 -> 67, 120 -> 60 on 3 x 100 x 110
    // (15 of 16) 85 -> 59.
    const bool padded = (g.c_in + 7) / 8 * 16 < (g.c_in + 31) / 32 * 4 * 15;
    if (waves < (mask_in || !padded ? 4096 : 1024) && f32_rounds(g, mask_in != nullptr)) return launch_f32_rounds(g, x, mask_in, mask_out, w, bias, idx, count, out, s);
    if (waves < (mask_in ? 4096 : 1024)) return FC_F32(32, 4, 6);
    return wide ? FC_F32(64, 1, 2) : FC_F32(32, 1, 3);
#undef FC_F32
}

// ---------------------------------------------------------------------------------------------
// Grouped layers of 16-bit storage.  Bound: HBM / L2 (x read, out written).
//
// An output channel's products hold its own group's inputs and nothing else: a foreign input times a
// zero weight would be NaN where that input is infinite or NaN.
//
// 16 channels per group and more (k_conv_grouped): a wave owns 16 output channels of one group.  The
// reduction is taps x input channels of the group, cut into pieces of 8 channels of one tap; four pieces
// make one v_mfma_f32_16x16x32: lane (column, quarter) holds piece 4 s + quarter, for the weights of output
// channel `column` and for the pixel of position `column`.  The weights of the block stay in registers for all
// rows of the span; a row tile is 16 positions, its loads issued a tile ahead.  The four waves of a workgroup
// take neighbouring channel blocks.
//
// 4 or 8 channels per group (k_conv_grouped_quads): v_mfma_f32_4x4x4_16b multiplies sixteen independent 4 x 4
// blocks.  A block is four output channels of one group at four positions, so a wave covers 64 channels of
// four positions per instruction and 4 input channels of one tap; lane (block, j) holds output
// channel 4 block + j of the weights and position j of the pixels, and ends with its block's four channels
// at position j.  Nothing is multiplied for padding, and the rate (1/4 of the large instructions') is still far
// from being the bound: 4 -> 4 channels on 16 x 56 x 56, half kept, is 0.4 us of them.  The halves of an
// 8-channel piece are summed apart and added at the end (as one chain the error of 8 -> 8 f16 channels against 64-bit
// sums is 7.4e-8 of the result, so 6.1e-8; products of 32 elements had 5.8e-8).  The four waves of a workgroup take the
// quads of rows in turn.  (8 -> 8 in the window form below: two products of 16 channels instead.)
// (With a mask / without one / with a list and no zero-fill, us, when this form was chosen: 128 channels in 32 groups on 16 x 56 x 56 12.6 / 12.8 /
// 13.1, and at stride 2 9.2 / 8.4 / 8.8; 256 in 32 groups 21.8 / 24.4 / 23.0.  16-channel products with zero weights for the
// foreign groups, which mixed groups as said above: 12.9 / 13.8 / 15.0, 10.0 / 9.6 / 9.9, 22.8 / 23.8 / 26.2.  On the vector
// ALUs, with a compaction and a zero-fill launch, the first of these was 61 us.)
// ---------------------------------------------------------------------------------------------
template <int DT>
__device__ __forceinline__ f32x4_t mfma16(const u32x4_t &a, const u32x4_t &b, const f32x4_t &c)
{
    if constexpr (DT == FC_BF16)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c,
                                                       0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0,
                                                      0, 0);
}

// sixteen independent products of 4 x 4 x 4: lane (block, j) holds row j of `a` and column j of `b`, four elements each
template <int DT>
__device__ __forceinline__ f32x4_t mfma4(const uint2 &a, const uint2 &b, const f32x4_t &c)
{
    if constexpr (DT == FC_BF16) {
        typedef short i16x4_t __attribute__((ext_vector_type(4)));
        return __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_bit_cast(i16x4_t, a), __builtin_bit_cast(i16x4_t, b), c, 0, 0, 0);
    } else {
        typedef _Float16 f16x4_t __attribute__((ext_vector_type(4)));
        return __builtin_amdgcn_mfma_f32_4x4x4f16(__builtin_bit_cast(f16x4_t, a), __builtin_bit_cast(f16x4_t, b), c, 0, 0, 0);
    }
}

__device__ __forceinline__ void relu4(f32x4_t &v)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = !(v[i] > 0.f) ? (v[i] != v[i] ? v[i] : 0.f) : v[i];
}

// g: the whole layer (all groups); cig / cog: channels of one group; KS: matrix steps
template <int DT, typename TO, int KS>
__global__ __launch_bounds__(kRegThreads, KS > 9 ? 1 : 2) void k_conv_grouped(
    Geom g, int cig, int cog, const uint16_t *__restrict__ x, const uint8_t *__restrict__ mask_in,
    const uint8_t *__restrict__ mask_out, const uint16_t *__restrict__ w, const float *__restrict__ bias,
    const int32_t *__restrict__ idx, const int32_t *__restrict__ count, TO *__restrict__ out)
{
    constexpr int S = kGroupedSpan;
    __shared__ SpanRows rows_s;
    const int rows = idx ? *count : g.m;
    const int first = blockIdx.x * S;
    if (first >= rows) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, col = lane & 15, quarter = lane >> 4;
    const int co0 = (blockIdx.y * 4 + wave) * 16;
    const int taps = g.kh * g.kw;
    const int win0 = (co0 / cog) * cig; // first input channel of the block's group
    const int ppt = cig >> 3;           // pieces per tap

    // this lane's part of the block's weights, and where its pieces lie in a pixel's neighbourhood
    // (loaded first: they are on their way while the rows are set up)
    const __amdgpu_buffer_rsrc_t rw =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(w), 0, (uint32_t)g.c_out * taps * cig * 2u, 0x00020000);
    u32x4_t wf[KS];
    uint32_t xo[KS];  // byte offset of the piece from the row's first tap (of tensors of up to 0xF0000000 bytes)
    uint32_t xsel[KS];// its tap's bit
    {
        const int co = co0 + col;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int q = s * 4 + quarter;
            const int tap = (int)((uint32_t)q / (uint32_t)ppt), pc = q - tap * ppt;
            const int kh = (int)((uint32_t)tap / (uint32_t)g.kw), kw = tap - kh * g.kw;
            xo[s] = (uint32_t)((kh * g.dh * g.w + kw * g.dw) * g.c_in + win0 + pc * 8) * 2u;
            xsel[s] = tap < taps ? 1u << tap : 0u;
            wf[s] = __builtin_amdgcn_raw_buffer_load_b128(
                rw, tap < taps && co < g.c_out ? (uint32_t)((co * taps + tap) * cig + pc * 8) * 2u : kOutOfRange, 0, 0);
        }
    }
    int n, nd;
    span_rows<S>(g, mask_in, mask_out, idx, rows, first, rows_s, &n, &nd);
    if (nd && !(g.flags & FC_SKIP_ZERO_FILL))
        clear_dropped<TO>(rows_s, nd, out, g.c_out, blockIdx.y * 64, min(64, g.c_out - (int)blockIdx.y * 64));
    if (co0 >= g.c_out) return; // (nothing below waits for this wave)

    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t *>(x), 0, (uint32_t)g.n * g.h * g.w * g.c_in * 2u, 0x00020000);
    float4 bq = make_float4(0.f, 0.f, 0.f, 0.f);
    if (bias) bq = *reinterpret_cast<const float4 *>(bias + co0 + quarter * 4);
    u32x4_t xv[2][KS];
    auto load = [&](auto set_c, int r) __attribute__((always_inline)) {
        constexpr int st = decltype(set_c)::value;
        const bool live = r < n; // (n <= kMaxSpan; r may point past it)
        const uint32_t base = live ? (uint32_t)rows_s.base[r] * (uint32_t)g.c_in * 2u : 0u; // (modulo 2^32 until xo is added)
        const uint32_t bits = live ? rows_s.bits[0][r] : 0u;
#pragma unroll
        for (int s = 0; s < KS; ++s)
            xv[st][s] = __builtin_amdgcn_raw_buffer_load_b128(rx, (bits & xsel[s]) ? base + xo[s] : kOutOfRange,
                                                              0, 0);
    };
    auto multiply = [&](auto set_c, int r) __attribute__((always_inline)) {
        constexpr int st = decltype(set_c)::value;
        f32x4_t acc = {bq.x, bq.y, bq.z, bq.w};
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < KS; ++s) acc = mfma16<DT>(wf[s], xv[st][s], acc);
        if (g.flags & FC_RELU) relu4(acc);
        if (r < n)
            store4<DT, TO>(out + (int64_t)rows_s.p[r] * g.c_out + co0 + quarter * 4, acc[0], acc[1], acc[2], acc[3]);
    };
    using C0 = std::integral_constant<int, 0>;
    using C1 = std::integral_constant<int, 1>;
    // (tiles past the end load nothing but are issued all the same, see k_conv_f32)
    load(C0{}, col);
    for (int r = col; r - col < n; r += 32) {
        load(C1{}, r + 16);
        multiply(C0{}, r);
        if (r - col + 16 >= n) break;
        load(C0{}, r + 32);
        multiply(C1{}, r + 16);
    }
}

// 4 or 8 channels per group.  A lane's weights are one run of taps x cig elements (channel blk0 + lane), staged with the
// workgroup's other channels as one block through LDS; its pixels are taps x cig elements in loads of V
// times four channels: NL >= taps * cig / (4 V) loads (NL = 9: cig = 4 V only).
template <int DT, typename TO, int V, int NL>
__global__ __launch_bounds__(kRegThreads, V * NL > 36 ? 1 : 2) void k_conv_grouped_quads(
    Geom g, int cig, int cog, const uint16_t *__restrict__ x, const uint8_t *__restrict__ mask_in,
    const uint8_t *__restrict__ mask_out, const uint16_t *__restrict__ w, const float *__restrict__ bias,
    const int32_t *__restrict__ idx, const int32_t *__restrict__ count, TO *__restrict__ out)
{
    constexpr int S = kGroupedSpan;
    constexpr int NB = V * NL > 36 ? 1 : 2; // quads whose pixels are held
    constexpr bool ONE = NL == 9;           // one load per tap (cig == 4 V)
    extern __shared__ __align__(16) unsigned char lds[]; // weights
    __shared__ SpanRows rows_s;
    const int rows = idx ? *count : g.m;
    const int first = blockIdx.x * S;
    if (first >= rows) return;
    const int tid = threadIdx.x, lane = tid & 63, j = lane & 3, blk0 = blockIdx.y * 64;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int taps = g.kh * g.kw;
    // byte offsets of the taps, kept in scalar registers where a tap is one load (what a quad costs is the instructions
    // of its addresses)
    uint32_t tap_at[ONE ? NL : 1];
    if constexpr (ONE) {
        int kw = 0;
        uint32_t row = 0;
#pragma unroll
        for (int s = 0; s < NL; ++s) {
            tap_at[s] = s < taps ? row + (uint32_t)(kw * g.dw * g.c_in) * 2u : 0u;
            if (++kw == g.kw) {
                kw = 0;
                row += (uint32_t)(g.dh * g.w * g.c_in) * 2u;
            }
        }
    }
    {
        const u32x4_t rsrc_w = make_rsrc_words(w, (uint32_t)g.c_out * taps * cig * 2u);
        const uint32_t at = (uint32_t)(blk0 * taps * cig) * 2u, bytes = (uint32_t)(64 * taps * cig) * 2u;
        const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>(lds);
        for (uint32_t o = (uint32_t)wave * 1024u; o < bytes; o += 4096u) // (the block's size is rounded up to 1 KB)
            dma_load16(rsrc_w, at + o + (uint32_t)lane * 16u, __builtin_amdgcn_readfirstlane(lds0 + o));
    }
    int n, nd;
    span_rows<S>(g, mask_in, mask_out, idx, rows, first, rows_s, &n, &nd);
    if (nd && !(g.flags & FC_SKIP_ZERO_FILL))
        clear_dropped<TO>(rows_s, nd, out, g.c_out, blk0, min(64, g.c_out - blk0));
    wait_vmcnt<0>();
    __syncthreads();
    if (n == 0) return;

    const int co = blk0 + (lane & ~3); // the block's channels co .. co + 3, all of one group
    uint2 wf[NL][V];
#pragma unroll
    for (int s = 0; s < NL; ++s)
#pragma unroll
        for (int v = 0; v < V; ++v)
            wf[s][v] = s * V * 4 < taps * cig ? *reinterpret_cast<const uint2 *>(lds + (lane * taps * cig + (s * V + v) * 4) * 2)
                                              : make_uint2(0u, 0u);
    // (x through a descriptor that starts a padding's worth earlier, see k_conv_f32: a tap's offset is then a scalar)
    const uint32_t xbias = (uint32_t)(g.ph * g.w + g.pw) * (uint32_t)g.c_in * 2u;
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t *>(x) - xbias / 2, 0, (uint32_t)g.n * g.h * g.w * g.c_in * 2u + xbias, 0x00020000);
    float4 bq = make_float4(0.f, 0.f, 0.f, 0.f);
    if (bias && co < g.c_out) bq = *reinterpret_cast<const float4 *>(bias + co);
    // Pixels are loaded with neighbouring lanes on neighbouring channels - lane 16 row + block, whole lines of four rows
    // (lanes 4 block + row, as the products take them, are 64 lines to the address unit: 22.0 us for 4 -> 4 channels on 16 x 56 x 56, half kept, where this takes 13.1)
    // - and change lanes on their way to the product.
    const int load_block = lane & 15, load_co = blk0 + load_block * 4;
    const uint32_t group_off = (uint32_t)(load_co / cog * cig) * 2u;
    const int from_lane = (j * 16 + (lane >> 2)) * 4;
    auto to_block = [&](const uint2 &v) __attribute__((always_inline)) {
        return make_uint2((uint32_t)__builtin_amdgcn_ds_bpermute(from_lane, (int)v.x),
                          (uint32_t)__builtin_amdgcn_ds_bpermute(from_lane, (int)v.y));
    };
    uint2 xv[NB][NL][V];
    auto load = [&](auto set_c, int quad) __attribute__((always_inline)) {
        constexpr int st = decltype(set_c)::value;
        const int r = quad + (lane >> 4);
        const bool live = r < n && load_co < g.c_out; // (n <= kMaxSpan; r may point past it)
        const uint32_t base = live ? (uint32_t)rows_s.base[r] * (uint32_t)g.c_in * 2u + xbias + group_off : 0u;
        const uint32_t bits = live ? rows_s.bits[0][r] : 0u;
        auto fetch = [&](int s, int tap, uint32_t at) __attribute__((always_inline)) {
            const uint32_t on = tap < taps ? (uint32_t)__builtin_amdgcn_sbfe((int)bits, (uint32_t)tap, 1) : 0u;
            const uint32_t off = (base & on) | (kOutOfRange & ~on);
            if constexpr (V == 1) {
                const auto t = __builtin_amdgcn_raw_buffer_load_b64(rx, off, at, 0);
                xv[st][s][0] = make_uint2(t[0], t[1]);
            } else {
                const auto t = __builtin_amdgcn_raw_buffer_load_b128(rx, off, at, 0);
                xv[st][s][0] = make_uint2(t[0], t[1]);
                xv[st][s][1] = make_uint2(t[2], t[3]);
            }
        };
        if constexpr (ONE) {
#pragma unroll
            for (int s = 0; s < NL; ++s) fetch(s, s, tap_at[s]);
        } else {
            int tap = 0, kw = 0, sub = 0; // of the load (the same for all lanes)
            uint32_t row = 0;             // byte offset of the tap's kernel row
#pragma unroll
            for (int s = 0; s < NL; ++s) {
                fetch(s, tap, tap < taps ? row + (uint32_t)(kw * g.dw * g.c_in + sub) * 2u : 0u);
                sub += 4 * V;
                if (sub == cig) {
                    sub = 0;
                    ++tap;
                    if (++kw == g.kw) {
                        kw = 0;
                        row += (uint32_t)(g.dh * g.w * g.c_in) * 2u;
                    }
                }
            }
        }
    };
    auto multiply = [&](auto set_c, int quad) __attribute__((always_inline)) {
        constexpr int st = decltype(set_c)::value;
        const int r = quad + j;
        f32x4_t sum[2] = {{bq.x, bq.y, bq.z, bq.w}, {0.f, 0.f, 0.f, 0.f}};
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < NL; ++s)
#pragma unroll
            for (int v = 0; v < V; ++v) sum[v] = mfma4<DT>(wf[s][v], to_block(xv[st][s][v]), sum[v]);
        f32x4_t acc = V == 1 ? sum[0] : sum[0] + sum[1];
        if (g.flags & FC_RELU) relu4(acc);
        if (r < n && co < g.c_out) store4<DT, TO>(out + (int64_t)rows_s.p[r] * g.c_out + co, acc[0], acc[1], acc[2], acc[3]);
    };
    using C0 = std::integral_constant<int, 0>;
    using C1 = std::integral_constant<int, NB - 1>;
    const int r0 = wave * 4; // wave v: quads v, v + 4, ...
    if constexpr (NB == 1) {
        for (int r = r0; r < n; r += 16) {
            load(C0{}, r);
            multiply(C0{}, r);
        }
    } else {
        load(C0{}, r0);
        for (int r = r0; r < n; r += 32) {
            load(C1{}, r + 16);
            multiply(C0{}, r);
            if (r + 16 >= n) break;
            load(C0{}, r + 32);
            multiply(C1{}, r + 16);
        }
    }
}

// The same layers where output positions are input pixels (unit stride, same size) and there is no list.
// The kernels above spend much of their time on addresses and on waiting for gathers one quad or tile ahead.
// Here the pixels under a span of 64 consecutive positions are, for every kernel row, one run of
// 64 + (kw - 1) dil_w consecutive pixels: they are staged in LDS once (whole 128-byte pieces of 64 output
// channels' groups), the workgroup's weights likewise, and all operands come from there; a gated tap
// reads a piece of zeros.  V = 0: blocks of 16 channels, KS matrix steps; NG = 2: a block of two groups of 8, a product for each
// on the same weights, of which every lane keeps its own group's rows (256 channels in 32 groups on 16 x 56 x 56: 21.8 us with half
// the pixels kept and 24.4 without a mask, now 19.8 and 23.7, as quads 22.4 and 25.2: those read a pixel's pieces twice).  V = 1, 2: quads of rows, 3x3 kernels and 4 V
// input channels per group, so that a tap is one read; everything about the reads is fixed when the kernel is compiled
// (a pixel's pieces 1 << LG, its kernel row's line), because what a quad costs is the instructions of its addresses: with
// the line's length and the taps at run time the kernel took 17.8 us where it then took 12.5 and now takes 11.8 (4 -> 4 channels on 16 x 56 x 56, half kept).
constexpr int kWindowSpan = 64;
constexpr int kQuadLine = kWindowSpan + 4; // pixel slots of a line: one of zeros, 66 pixels, one to make four divide it
struct WindowCut {
    int32_t line;      // pixels of a kernel row's run
    int32_t lg_pieces; // log2 of the 16-byte pieces of a pixel's window
    int32_t x_bytes, w_bytes;
    FastDiv by_line, by_kw, by_ppt;
    // of the workgroups: the 64-channel blocks of a span in a row or, block_major, the spans of a block; see xcd_eighth_of
    FastDiv by_inner;
    uint32_t inner : 26, lg_order : 5, block_major : 1;
};

template <int DT, typename TO, int V, int KS, int LG, int NG = 1>
__global__ __launch_bounds__(kRegThreads, 2) void k_conv_grouped_window(
    Geom g, WindowCut cut, int cig, int cog, const uint16_t *__restrict__ x, const uint8_t *__restrict__ mask_in,
    const uint8_t *__restrict__ mask_out, const uint16_t *__restrict__ w, const float *__restrict__ bias,
    TO *__restrict__ out)
{
    // [pixels | weights | 16 bytes of zeros | tap bits | kept positions, then dropped ones from the end]
    extern __shared__ __align__(16) unsigned char lds[];
    unsigned char *w_s = lds + cut.x_bytes, *zero_s = w_s + cut.w_bytes;
    uint32_t *bits_s = reinterpret_cast<uint32_t *>(zero_s + 16);
    uint8_t *order_s = reinterpret_cast<uint8_t *>(bits_s + kWindowSpan);
    const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>(lds);
    const int tid = threadIdx.x, lane = tid & 63, col = lane & 15, quarter = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int span, blk;
    if (cut.block_major == 0) {
        const int unit = xcd_eighth((int)blockIdx.x, (int)gridDim.x);
        span = (int)fast_div((uint32_t)unit, cut.by_inner), blk = unit - span * (int)cut.inner;
    } else {
        const int unit = xcd_eighth_of((int)blockIdx.x, (int)gridDim.x, (int)cut.lg_order);
        blk = (int)fast_div((uint32_t)unit, cut.by_inner), span = unit - blk * (int)cut.inner;
    }
    const int first = span * kWindowSpan, blk0 = blk * 64, co0 = blk0 + wave * 16;
    const int taps = g.kh * g.kw;
    const int win0 = (blk0 / cog) * cig; // first input channel of the workgroup's groups
    const int lg_pieces = V ? LG : cut.lg_pieces, line = V ? kQuadLine : cut.line;
    // Sixteen lanes that read one piece of sixteen neighbouring pixels, or a few pieces each of the four pixels of a quad,
    // meet in different banks (two pixels of 128 bytes, or one of 256, fill all of them).
    auto swizzle = [&](int q) { return V == 0 ? q >> 1 : (LG == 4 ? q : q >> 1) << 2; };

    // ---- weights: one contiguous block ----
    {
        const u32x4_t rsrc_w = make_rsrc_words(w, (uint32_t)g.c_out * taps * cig * 2u);
        const uint32_t at = (uint32_t)(blk0 * taps * cig) * 2u;
        for (uint32_t o = (uint32_t)wave * 1024u; o < (uint32_t)cut.w_bytes; o += 4096u)
            dma_load16(rsrc_w, at + o + (uint32_t)lane * 16u, __builtin_amdgcn_readfirstlane(lds0 + cut.x_bytes + o));
    }
    // ---- pixels: LDS piece c of pixel slot q holds the window's piece c ^ swizzle(q).  (A pixel before or past its image may be another image's or,
    // checked by the descriptor, none: no tap reads it.) ----
    const u32x4_t rsrc_x = make_rsrc_words(x, (uint32_t)g.n * g.h * g.w * g.c_in * 2u);
    const int pieces = 1 << lg_pieces, slots = g.kh * line;
    auto pixel_at = [&](int o) __attribute__((always_inline)) {
        const int i = o + lane, q = i >> lg_pieces, c = (i ^ swizzle(q)) & (pieces - 1);
        const int k = V ? (int)((uint32_t)q / (uint32_t)kQuadLine) : (int)fast_div((uint32_t)q, cut.by_line);
        const int t = q - k * line - (V ? 1 : 0), ch = win0 + c * 8;
        const int pix = first + (k * g.dh - g.ph) * g.w - g.pw + t;
        return (V == 0 || t >= 0) && q < slots && ch < g.c_in ? ((uint32_t)pix * (uint32_t)g.c_in + (uint32_t)ch) * 2u : kOutOfRange;
    };
    auto request_pixels = [&]() __attribute__((always_inline)) {
        for (int o = wave * 64; o < (slots << lg_pieces); o += kRegThreads)
            dma_load16(rsrc_x, pixel_at(o), __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)o * 16u));
    };
    if (!mask_in) request_pixels();
    // ---- labels: lane l of every wave holds position first + l; they and the mask under this wave's share of the taps are requested together
    // (one after another they were four round trips), and while they are on their way a quad kernel finds its pixels' addresses.  4 -> 4
    // channels on 16 x 56 x 56, half kept, 13.4 -> 11.8 us, 8 -> 8 there 21.6 -> 19.8, 16 -> 16 on 32 x 60 x 60 48.9 -> 45.3. ----
    const int p = first + lane;
    const bool inside = p < g.m, packed = (g.flags & FC_PACKED_MASKS) != 0;
    const int pp = inside ? p : 0;
    const int r = (int)fast_div((uint32_t)pp, g.div_wo), ow = pp - r * g.wo;
    const int img = (int)fast_div((uint32_t)r, g.div_ho), oh = r - img * g.ho;
    constexpr int U = 3; // look-ups in flight
    bool in[U];
    int tap_pix[U];
    uint32_t m[U + 1]; // and the label
    auto tap_places = [&](int t0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int t = t0 + 4 * u, kh = (int)fast_div((uint32_t)t, cut.by_kw), kw = t - kh * g.kw;
            const int ih = oh - g.ph + kh * g.dh, iw = ow - g.pw + kw * g.dw;
            in[u] = inside && t < taps && (uint32_t)ih < (uint32_t)g.h && (uint32_t)iw < (uint32_t)g.w;
            tap_pix[u] = in[u] ? (img * g.h + ih) * g.w + iw : 0;
            m[u] = 1u;
        }
    };
    tap_places(wave);
    constexpr int PL = V ? ((3 * kQuadLine << LG) + kRegThreads - 1) / kRegThreads : 1; // quads: a lane's pieces
    uint32_t from[PL];
    m[U] = 1u;
    if (mask_in) {
        const int ihc = min(max(oh - g.ph + g.dh * ((g.kh - 1) / 2), 0), g.h - 1), iwc = min(max(ow - g.pw + g.dw * ((g.kw - 1) / 2), 0), g.w - 1);
        m[U] = mask_at(mask_out ? mask_out : mask_in, mask_out ? pp : (img * g.h + ihc) * g.w + iwc, packed);
#pragma unroll
        for (int u = 0; u < U; ++u) m[u] = mask_at(mask_in, tap_pix[u], packed);
        if constexpr (V != 0) {
#pragma unroll
            for (int i = 0; i < PL; ++i) from[i] = pixel_at(wave * 64 + i * kRegThreads);
        }
        loaded_together(m);
    }
    const bool kept = inside && m[U];
    const uint64_t kept_set = __ballot(kept), drop_set = __ballot(inside && !kept);
    const int n = __popcll(kept_set), nd = __popcll(drop_set);
    if (mask_in && n > 0) {
        if constexpr (V != 0) {
#pragma unroll
            for (int i = 0; i < PL; ++i) {
                const int o = wave * 64 + i * kRegThreads;
                if (o < (slots << LG)) dma_load16(rsrc_x, from[i], __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)o * 16u));
            }
        } else {
            request_pixels();
        }
    }
    if (wave == 0) {
        const uint64_t below = (1ull << lane) - 1ull;
        if (kept) order_s[__popcll(kept_set & below)] = (uint8_t)lane;
        if (inside && !kept) order_s[kWindowSpan - 1 - __popcll(drop_set & below)] = (uint8_t)lane;
        bits_s[lane] = 0u;
        if (lane < 4) reinterpret_cast<uint32_t *>(zero_s)[lane] = 0u;
    }
    if (n > 0) {
        // ---- taps in use: this wave's share of them, for all positions ----
        __syncthreads(); // bits_s cleared
        uint32_t mine = 0;
        for (int t0 = wave; t0 < taps; t0 += 4 * U) {
            if (t0 != wave) {
                tap_places(t0);
                if (mask_in) {
#pragma unroll
                    for (int u = 0; u < U; ++u) m[u] = mask_at(mask_in, tap_pix[u], packed);
                    loaded_together(m);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) mine |= kept && in[u] && m[u] ? 1u << (t0 + 4 * u) : 0u;
        }
        if (mine) atomicOr(&bits_s[lane], mine);
    }
    wait_vmcnt<0>();
    __syncthreads();
    if (nd > 0 && !(g.flags & FC_SKIP_ZERO_FILL)) {
        const int pieces = min(64, g.c_out - blk0) * (int)sizeof(TO) / 16; // (16 divides the channels)
        const u32x4_t zero = {0u, 0u, 0u, 0u};
        for (int i = tid; i < nd * pieces; i += kRegThreads) {
            const int k = (int)((uint32_t)i / (uint32_t)pieces), c = i - k * pieces;
            const int64_t row = (int64_t)(first + order_s[kWindowSpan - 1 - k]) * g.c_out + blk0;
            __builtin_nontemporal_store(zero, reinterpret_cast<u32x4_t *>(out + row) + c);
        }
    }
    if (n == 0) return;
    const uint32_t pmask = (1u << lg_pieces) - 1u;
    if constexpr (V == 0) {
        const uint32_t zero_at = (uint32_t)(cut.x_bytes + cut.w_bytes);
        if (co0 >= g.c_out) return;
        // ---- this wave's 16 channels: weights from LDS to registers, and where their pieces lie ----
        const int ppt = cig >> 3;
        const int bw0 = (co0 / cog) * cig; // first input channel of the block's first group
        const int co = co0 + col;
        u32x4_t wf[KS];    // of the channel's own group
        int xq[KS];        // pixel slot of the piece from the position's own slot
        uint32_t xc[KS], xsel[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int q = s * 4 + quarter;
            const int tap = (int)fast_div((uint32_t)q, cut.by_ppt), pc = q - tap * ppt;
            const int kh = (int)fast_div((uint32_t)tap, cut.by_kw), kw = tap - kh * g.kw;
            xq[s] = kh * cut.line + kw * g.dw;
            xc[s] = (uint32_t)((bw0 - win0) >> 3) + (uint32_t)pc;
            xsel[s] = tap < taps ? 1u << tap : 0u;
            const u32x4_t zero = {0u, 0u, 0u, 0u};
            wf[s] = tap < taps ? *reinterpret_cast<const u32x4_t *>(w_s + (((co - blk0) * taps + tap) * cig + pc * 8) * 2) : zero;
        }
        float4 bq = make_float4(0.f, 0.f, 0.f, 0.f);
        if (bias) bq = *reinterpret_cast<const float4 *>(bias + co0 + quarter * 4);
        for (int r0 = 0; r0 < n; r0 += 16) {
            const bool live = r0 + col < n;
            const int j = live ? order_s[r0 + col] : 0;
            const uint32_t bits = live ? bits_s[j] : 0u;
            // a product per group: rows of the other group come out as anything and are dropped
            u32x4_t xv[NG][KS];
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const uint32_t q = (uint32_t)(j + xq[s]);
#pragma unroll
                for (int k = 0; k < NG; ++k) {
                    const uint32_t c = xc[s] + (uint32_t)(k * ppt);
                    const uint32_t at = ((q << cut.lg_pieces) + ((c ^ (uint32_t)swizzle((int)q)) & pmask)) * 16u;
                    xv[k][s] = *reinterpret_cast<const u32x4_t *>(lds + ((bits & xsel[s]) ? at : zero_at));
                }
            }
            f32x4_t of[NG];
#pragma unroll
            for (int k = 0; k < NG; ++k) {
                of[k] = f32x4_t{bq.x, bq.y, bq.z, bq.w};
#pragma unroll
                for (int s = 0; s < KS; ++s) of[k] = mfma16<DT>(wf[s], xv[k][s], of[k]);
            }
            f32x4_t acc;
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] = NG == 1 || quarter < 2 ? of[0][i] : of[NG - 1][i];
            if (g.flags & FC_RELU) relu4(acc);
            if (live)
                store4<DT, TO>(out + (int64_t)(first + j) * g.c_out + co0 + quarter * 4, acc[0], acc[1], acc[2], acc[3]);
        }
    } else {
        // ---- lane (block, j): the weights of channel blk0 + lane, and the pixels of row j of a quad ----
        constexpr uint32_t PIX = 16u << LG, LINE = kQuadLine * PIX; // bytes
        const int j = lane & 3, co = blk0 + (lane & ~3);
        uint2 wf[9][V];
#pragma unroll
        for (int s = 0; s < 9; ++s)
#pragma unroll
            for (int v = 0; v < V; ++v) wf[s][v] = *reinterpret_cast<const uint2 *>(w_s + (lane * 9 + s) * 8 * V + v * 8);
        float4 bq = make_float4(0.f, 0.f, 0.f, 0.f);
        if (bias && co < g.c_out) bq = *reinterpret_cast<const float4 *>(bias + co);
        const uint32_t in_pixel = (uint32_t)((co / cog) * cig - win0) * 2u; // the block's group in a pixel
        TO *const o = out + (int64_t)first * g.c_out + co;
        // wave v: quads v, v + 4, ... of the kept rows
        int row[kWindowSpan / 16];
        uint32_t bits[kWindowSpan / 16];
#pragma unroll
        for (int u = 0; u < kWindowSpan / 16; ++u) row[u] = order_s[wave * 4 + u * 16 + j];
#pragma unroll
        for (int u = 0; u < kWindowSpan / 16; ++u) {
            const bool live = wave * 4 + u * 16 + j < n && co < g.c_out;
            bits[u] = bits_s[row[u] & (kWindowSpan - 1)];
            row[u] = live ? row[u] : -1;
            bits[u] = live ? bits[u] : 0u;
        }
#pragma unroll
        for (int u = 0; u < kWindowSpan / 16; ++u) {
            if (wave * 4 + u * 16 >= n) break;
            // a tap that is off reads its line's slot of zeros
            uint2 xv[9][V];
#pragma unroll
            for (int kw = 0; kw < 3; ++kw) {
                const uint32_t q = (uint32_t)(row[u] + 1 + kw);
                const uint32_t at = q * PIX + (((in_pixel >> 4) ^ (uint32_t)swizzle((int)q)) & pmask) * 16u + (in_pixel & 15u);
#pragma unroll
                for (int kh = 0; kh < 3; ++kh) {
                    const uint32_t on = (uint32_t)__builtin_amdgcn_sbfe((int)bits[u], kh * 3 + kw, 1);
                    const unsigned char *from = lds + (at & on) + kh * LINE;
                    if constexpr (V == 1) {
                        xv[kh * 3 + kw][0] = *reinterpret_cast<const uint2 *>(from);
                    } else {
                        const uint4 t = *reinterpret_cast<const uint4 *>(from);
                        xv[kh * 3 + kw][0] = make_uint2(t.x, t.y);
                        xv[kh * 3 + kw][1] = make_uint2(t.z, t.w);
                    }
                }
            }
            f32x4_t sum[2] = {{bq.x, bq.y, bq.z, bq.w}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int s = 0; s < 9; ++s)
#pragma unroll
                for (int v = 0; v < V; ++v) sum[v] = mfma4<DT>(wf[s][v], xv[s][v], sum[v]);
            f32x4_t acc = V == 1 ? sum[0] : sum[0] + sum[1];
            if (g.flags & FC_RELU) relu4(acc);
            if (row[u] >= 0) store4<DT, TO>(o + row[u] * g.c_out, acc[0], acc[1], acc[2], acc[3]);
        }
    }
}

// The reduction of a 16-channel block, or of as many channels as make one, in 32-element steps: the measure of the weights
// a lane holds
static int grouped_steps(const Geom &g, int cig, int cog)
{
    const int ic = cog >= 16 ? cig : (16 / cog) * cig;
    return (g.kh * g.kw * (ic / 8) + 3) / 4;
}

bool conv_grouped_supported(const Geom &g, int groups, int in_dtype, int out_dtype)
{
    if (in_dtype != FC_BF16 && in_dtype != FC_F16) return false;
    if (out_dtype != in_dtype && out_dtype != FC_F32) return false;
    const int cig = g.c_in / groups, cog = g.c_out / groups;
    // quads of channels inside a group with whole 8-byte pieces of its inputs, or 16-channel blocks inside a group with
    // whole 16-byte pieces (one or two channels per group: a quad would mix groups, the direct kernel keeps them apart)
    if (g.c_out % 16 != 0 || g.c_in % 8 != 0 || cig % 4 != 0) return false;
    if (cog != 4 && cog != 8 && (cog % 16 != 0 || cig % 8 != 0)) return false;
    if (g.kh * g.kw > 32 || grouped_steps(g, cig, cog) > 18) return false; // tap bits; weights in registers
    if (g.h > 16384 || g.w > 16384 || g.ph > 8192 || g.pw > 8192) return false;
    // (quads read x through a descriptor that starts ph rows and pw pixels early)
    const uint64_t early = cog < 16 ? (uint64_t)g.ph * g.w + g.pw : 0;
    return ((uint64_t)g.n * g.h * g.w + early) * g.c_in * 2u < kBufferLimit &&
           (uint64_t)g.c_out * g.kh * g.kw * cig * 2u < kBufferLimit;
}

template <int DT, typename TO>
static hipError_t launch_grouped(const Geom &g, int groups, const void *x, const uint8_t *mask_in, const uint8_t *mask_out,
                                 const void *w, const float *bias, const int32_t *idx, const int32_t *count, void *out,
                                 hipStream_t s)
{
    const int cig = g.c_in / groups, cog = g.c_out / groups, taps = g.kh * g.kw, steps = grouped_steps(g, cig, cog);
    const bool quads = cog < 16;
    const int v = cig % 8 == 0 ? 2 : 1; // quads: 4-channel pieces of a load
    const bool pairs = cog == 8 && v == 2; // windows: two groups of a 16-channel block
    // spans of positions as windows of pixels: unit stride, same size, no list, groups that do not straddle a
    // workgroup's 64 channels and whose channels make a power of two of 16-byte pieces, at most 64 KB of LDS; quads: what
    // their form is compiled for
    const int wch = cog <= 64 && 64 % cog == 0 ? 64 / cog * cig : 0;
    if (!idx && g.sh == 1 && g.sw == 1 && g.ho == g.h && g.wo == g.w && wch >= 32 && wch <= 128 && (wch & (wch - 1)) == 0 &&
        (pairs || !quads ? steps <= 9 : g.kh == 3 && g.kw == 3 && g.dw == 1 && cig == 4 * v)) {
        WindowCut cut;
        cut.line = quads && !pairs ? kQuadLine : kWindowSpan + (g.kw - 1) * g.dw;
        cut.lg_pieces = wch == 32 ? 2 : (wch == 64 ? 3 : 4);
        cut.x_bytes = (g.kh * cut.line * wch * 2 + 1023) & ~1023;
        cut.w_bytes = (64 * taps * cig * 2 + 1023) & ~1023;
        cut.by_line = make_fastdiv((uint32_t)cut.line);
        cut.by_kw = make_fastdiv((uint32_t)g.kw);
        cut.by_ppt = make_fastdiv((uint32_t)(cig >= 8 ? cig / 8 : 1));
        const int bytes = cut.x_bytes + cut.w_bytes + 16 + kWindowSpan * 5;
        if (bytes <= 64 * 1024) {
            // (quads: 4 -> 8, 4 -> 4, 8 -> 4 channels per group)
            auto kern = pairs ? (taps * cig <= 96 ? k_conv_grouped_window<DT, TO, 0, 3, 0, 2> : k_conv_grouped_window<DT, TO, 0, 5, 0, 2>)
                        : !quads ? (steps <= 5 ? k_conv_grouped_window<DT, TO, 0, 5, 0> : k_conv_grouped_window<DT, TO, 0, 9, 0>)
                        : v == 1 ? (cog == 8 ? k_conv_grouped_window<DT, TO, 1, 9, 2> : k_conv_grouped_window<DT, TO, 1, 9, 3>)
                                 : k_conv_grouped_window<DT, TO, 2, 9, 4>;
            // Neighbouring windows share rows of pixels: an XCD takes an eighth of the work in one piece, spans with all their blocks.  With a mask and fewer images
            // than XCDs that piece may be all kept or all irrelevant.  Where the blocks are a multiple of eight an XCD then takes whole blocks; else eight spans at a
            // time.  us, as numbered -> eighths (-> by this rule, where it is another), masks of regions, other buffers each time: 128 channels in 32 groups on
            // 16 x 56 x 56 11.8 -> 11.1, without a mask 13.4 -> 12.8, 256 on 16 x 28 x 28 8.5 -> 7.9; 512 on 2 x 60 x 60 9.9 -> 11.0 -> 9.0, with the lower half of
            // both images irrelevant 9.1 -> 11.2 -> 7.7; 128 on 1 x 200 x 200 9.6 -> 10.9 -> 9.8, lower half 8.4 -> 10.9 -> 8.2, on 5 x 56 x 56 6.5 -> 6.2 -> 6.3; 64 in
            // 16 groups on 7 x 100 x 100, lower half, 7.9 -> 8.9 -> 8.2.  What loses: lower halves of as many images as XCDs (512 on 8 x 30 x 30 9.0 -> 9.4), 32 images
            // of a map no cache holds (512 on 60 x 60, without a mask, 102.5 -> 106; 94.6 -> 92.3 where it is read again).
            const int spans = (g.m + kWindowSpan - 1) / kWindowSpan, blocks = (g.c_out + 63) / 64;
            const bool few = mask_in && g.n < 8;
            if ((int64_t)spans * blocks >= 1 << 24) return hipErrorInvalidValue; // (2^32 threads; x would be past 16 GB)
            cut.block_major = few;
            cut.inner = few ? spans : blocks;
            cut.by_inner = make_fastdiv(cut.inner);
            cut.lg_order = few && blocks % 8 != 0 ? 6 : kOneSegment;
            hipLaunchKernelGGL(kern, dim3(spans * blocks), dim3(kRegThreads), bytes, s,
                               g, cut, cig, cog, (const uint16_t *)x, mask_in, mask_out, (const uint16_t *)w, bias, (TO *)out);
            return hipGetLastError();
        }
    }
    const dim3 grid((g.m + kGroupedSpan - 1) / kGroupedSpan, (g.c_out + 63) / 64);
    if (quads) {
        const int loads = taps * cig / (4 * v), bytes = (64 * taps * cig * 2 + 1023) & ~1023;
        const bool one = cig == 4 * v && loads <= 9;
        auto kern = v == 1 ? (one ? k_conv_grouped_quads<DT, TO, 1, 9>
                                         : (loads <= 36 ? k_conv_grouped_quads<DT, TO, 1, 36> : k_conv_grouped_quads<DT, TO, 1, 72>))
                           : (one ? k_conv_grouped_quads<DT, TO, 2, 9>
                                         : (loads <= 18 ? k_conv_grouped_quads<DT, TO, 2, 18> : k_conv_grouped_quads<DT, TO, 2, 36>));
        hipLaunchKernelGGL(kern, grid, dim3(kRegThreads), bytes, s, g, cig, cog, (const uint16_t *)x, mask_in, mask_out,
                           (const uint16_t *)w, bias, idx, count, (TO *)out);
        return hipGetLastError();
    }
    auto kern = steps <= 5 ? k_conv_grouped<DT, TO, 5> : (steps <= 9 ? k_conv_grouped<DT, TO, 9> : k_conv_grouped<DT, TO, 18>);
    hipLaunchKernelGGL(kern, grid, dim3(kRegThreads), 0, s, g, cig, cog, (const uint16_t *)x, mask_in, mask_out,
                       (const uint16_t *)w, bias, idx, count, (TO *)out);
    return hipGetLastError();
}

hipError_t launch_conv_grouped(const Geom &g, int groups, int in_dtype, int out_dtype, const void *x, const uint8_t *mask_in,
                               const uint8_t *mask_out, const void *w, const float *bias, const int32_t *idx,
                               const int32_t *count, void *out, hipStream_t s)
{
    if (in_dtype == FC_BF16)
        return out_dtype == FC_F32 ? launch_grouped<FC_BF16, float>(g, groups, x, mask_in, mask_out, w, bias, idx, count, out, s)
                                   : launch_grouped<FC_BF16, uint16_t>(g, groups, x, mask_in, mask_out, w, bias, idx, count, out, s);
    return out_dtype == FC_F32 ? launch_grouped<FC_F16, float>(g, groups, x, mask_in, mask_out, w, bias, idx, count, out, s)
                               : launch_grouped<FC_F16, uint16_t>(g, groups, x, mask_in, mask_out, w, bias, idx, count, out, s);
}

} // namespace fc
