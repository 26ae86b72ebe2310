// Focused convolution of fp32 storage (any channel counts from four on) and of grouped layers of 16-bit
// storage, on the matrix cores.
//
// Sec. III-A as everywhere: rows = kept positions, columns = output channels, reduction = taps
// x input channels, gated taps read as zero.  What these two layer types have in common is
// that the matrix cores are not the bottleneck that LDS staging exists for:
//   - fp32: v_mfma_f32_32x32x2_f32 runs at 1/16 of the 16-bit rate, so a wave needs three
//     16-byte loads per lane for every 512 cycles of matrix work; the L1 delivers that;
//   - grouped: a layer's multiplies are few (a ResNeXt stage: 0.24 GFLOP), its time is the
//     reading of x and the writing of out, and a 16-channel output block needs only the
//     channels of its own groups.
// No tile is staged, no barrier separates the steps of a reduction, and every wave runs ahead
// on its own loads.
//
// Rows.  A workgroup owns a span of consecutive positions.  Without a list it labels the span
// itself, compacts the kept positions in LDS and clears the rows of the others, so a masked call
// is one launch: no compaction before it, no zero-fill after it (they were 4 to 9 us and 4 to 5 us
// of launches around kernels that now take about as long).  With a list the span is a run of list
// entries, and the caller clears the irrelevant rows.
#include "fc_dma_util.hpp"
#include <type_traits>

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
        uint8_t rel[U];
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
        for (int u = 0; u < U; ++u) rel[u] = mask_in ? (uint8_t)mask_at(mask_in, max(pix[u], 0), packed) : (uint8_t)1;
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
// Measured (mask given, call included): 64 -> 64 on 2 x 60 x 80, half kept: 75.5 us on the vector ALUs
// with a compaction and a zero-fill launch, 15.6 us; 128 -> 128 on 8 x 120 x 120 without a mask: 320 us =
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
    const uint32_t xbias = (uint32_t)(g.ph * g.w + g.pw) * (uint32_t)g.c_in * 4u;
    const u32x4_t rsrc_x = make_rsrc_words(reinterpret_cast<const unsigned char *>(x) - xbias,
                                           (uint32_t)g.n * g.h * g.w * g.c_in * 4u + xbias);
    const u32x4_t rsrc_w = make_rsrc_words(w, (uint32_t)g.c_out * taps * g.c_in * 4u);
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
        woff[j] = co < g.c_out ? (uint32_t)(co * taps * g.c_in + piece * 4) * 4u : kOutOfRange;
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

    // a lane's quad (b, q) = channels co0 + 32 b + 8 q + 4 half .. + 3 of the position of row r
    const int r = wm * 32 + l32;
    const int64_t at = r < n ? (int64_t)rows_s.p[r] * g.c_out : -1;
    auto finish = [&](int b, int q, float4 v) __attribute__((always_inline)) {
        const int co = co0 + b * 32 + q * 8 + half * 4;
        float e[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (bias && co + i < g.c_out) e[i] += bias[co + i];
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

// four channels: one piece; 64 taps: the tap-valid bits of a row; 32-bit byte offsets into x and w; row
// origins in 16 bits
bool conv_f32_supported(const Geom &g)
{
    return g.c_in >= 4 && g.kh * g.kw <= 64 && g.h <= 16384 && g.w <= 16384 && g.ph <= 8192 && g.pw <= 8192 &&
           ((uint64_t)g.n * g.h * g.w + (uint64_t)g.ph * g.w + g.pw) * g.c_in * 4u < kBufferLimit &&
           (uint64_t)g.c_out * g.kh * g.kw * g.c_in * 4u < kBufferLimit;
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
    if (waves < (mask_in ? 4096 : 1024)) return FC_F32(32, 4, 6);
    return wide ? FC_F32(64, 1, 2) : FC_F32(32, 1, 3);
#undef FC_F32
}

// ---------------------------------------------------------------------------------------------
// Grouped layers of 16-bit storage.  Bound: HBM / L2 (x read, out written).
//
// A wave owns 16 output channels; the groups they belong to read a window of IC input channels
// (16 / cog groups of cig channels, or the one group the block lies in).  The reduction of the
// block is taps x IC, cut into pieces of 8 channels of one tap; four pieces make one
// v_mfma_f32_16x16x32: lane (column, quarter) holds piece 4 s + quarter, for the weights of output
// channel `column` (zero outside its own group: the block-diagonal part costs nothing but
// matrix slots, of which there are plenty) and for the pixel of position `column`.  The weights
// of the block stay in registers for all rows of the span; a row tile is 16 positions, its loads
// issued a tile ahead.  The four waves of a workgroup take neighbouring channel blocks, so
// that together they read whole 128-byte lines.
// (128 channels in 32 groups, 16 x 56 x 56, 48 % irrelevant: 49 us on the vector ALUs, 9 us
// of compaction and 5 us of zero-fill around it.)
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
    const int ic = cog >= 16 ? cig : (16 / cog) * cig; // channels of the block's window
    const int win0 = (co0 / cog) * cig;
    const int ppt = ic >> 3; // pieces per tap

    // this lane's part of the block's weights, and where its pieces lie in a pixel's neighbourhood
    // (loaded first: they are on their way while the rows are set up)
    const __amdgpu_buffer_rsrc_t rw =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(w), 0, (uint32_t)g.c_out * taps * cig * 2u, 0x00020000);
    u32x4_t wf[KS];
    int xo[KS];       // byte offset of the piece from the row's first tap
    uint32_t xsel[KS];// its tap's bit
    {
        const int co = co0 + col;
        const int wch = (co / cog) * cig; // first input channel of this output channel's group
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int q = s * 4 + quarter;
            const int tap = (int)((uint32_t)q / (uint32_t)ppt), pc = q - tap * ppt;
            const int kh = (int)((uint32_t)tap / (uint32_t)g.kw), kw = tap - kh * g.kw;
            xo[s] = ((kh * g.dh * g.w + kw * g.dw) * g.c_in + win0 + pc * 8) * 2;
            xsel[s] = tap < taps ? 1u << tap : 0u;
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) {
                const int local = win0 + pc * 8 + hf * 4 - wch;
                const bool ok = tap < taps && co < g.c_out && local >= 0 && local < cig;
                const auto v = __builtin_amdgcn_raw_buffer_load_b64(
                    rw, ok ? (uint32_t)((co * taps + tap) * cig + local) * 2u : kOutOfRange, 0, 0);
                wf[s][2 * hf] = v[0];
                wf[s][2 * hf + 1] = v[1];
            }
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
        const int base = live ? rows_s.base[r] * g.c_in * 2 : 0;
        const uint32_t bits = live ? rows_s.bits[0][r] : 0u;
#pragma unroll
        for (int s = 0; s < KS; ++s)
            xv[st][s] = __builtin_amdgcn_raw_buffer_load_b128(rx, (bits & xsel[s]) ? (uint32_t)(base + xo[s]) : kOutOfRange,
                                                              0, 0);
    };
    auto multiply = [&](auto set_c, int r) __attribute__((always_inline)) {
        constexpr int st = decltype(set_c)::value;
        f32x4_t acc = {bq.x, bq.y, bq.z, bq.w};
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < KS; ++s) acc = mfma16<DT>(wf[s], xv[st][s], acc);
        if (g.flags & FC_RELU)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] = !(acc[i] > 0.f) ? (acc[i] != acc[i] ? acc[i] : 0.f) : acc[i];
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

// The same layer where output positions are input pixels (unit stride, same size) and there is no list.
// The kernel above spends most of its time on addresses: a lane's pieces lie in other lines than its
// neighbours', 64 cycles of the address unit per load, for the weights of a block as for the pixels.
// Here the pixels under a span of 64 consecutive positions are, for every kernel row, one run of
// 64 + (kw - 1) dil_w consecutive pixels: they are staged in LDS once (whole 128-byte pieces of 64 output
// channels' groups), the workgroup's weights likewise, and all operands come from there; a gated tap
// reads a piece of zeros.  (128 channels in 32 groups on 16 x 56 x 56, half kept: 16.6 us above.)
constexpr int kWindowSpan = 64;
struct WindowCut {
    int32_t line;      // pixels of a kernel row's run
    int32_t lg_pieces; // log2 of the 16-byte pieces of a pixel's window
    int32_t x_bytes, w_bytes;
    FastDiv by_line, by_kw, by_ppt;
};

template <int DT, typename TO, int KS>
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
    const int first = blockIdx.x * kWindowSpan, blk0 = blockIdx.y * 64, co0 = blk0 + wave * 16;
    const int taps = g.kh * g.kw;
    const int win0 = (blk0 / cog) * cig; // first input channel of the workgroup's groups

    // ---- weights: one contiguous block ----
    {
        const u32x4_t rsrc_w = make_rsrc_words(w, (uint32_t)g.c_out * taps * cig * 2u);
        const uint32_t at = (uint32_t)(blk0 * taps * cig) * 2u;
        for (uint32_t o = (uint32_t)wave * 1024u; o < (uint32_t)cut.w_bytes; o += 4096u)
            dma_load16(rsrc_w, at + o + (uint32_t)lane * 16u, __builtin_amdgcn_readfirstlane(lds0 + cut.x_bytes + o));
    }
    // ---- labels: lane l of every wave holds position first + l ----
    const int p = first + lane;
    const bool inside = p < g.m;
    const bool kept = inside && (!mask_in || position_kept(g, mask_in, mask_out, p));
    const uint64_t kept_set = __ballot(kept), drop_set = __ballot(inside && !kept);
    const int n = __popcll(kept_set), nd = __popcll(drop_set);
    if (wave == 0) {
        const uint64_t below = (1ull << lane) - 1ull;
        if (kept) order_s[__popcll(kept_set & below)] = (uint8_t)lane;
        if (inside && !kept) order_s[kWindowSpan - 1 - __popcll(drop_set & below)] = (uint8_t)lane;
        bits_s[lane] = 0u;
        if (lane < 4) reinterpret_cast<uint32_t *>(zero_s)[lane] = 0u;
    }
    if (n > 0) {
        // ---- pixels: LDS piece c of pixel slot q holds the window's piece c ^ (q >> 1) ----
        const int pieces = 1 << cut.lg_pieces;
        const u32x4_t rsrc_x = make_rsrc_words(x, (uint32_t)g.n * g.h * g.w * g.c_in * 2u);
        const int npix = g.n * g.h * g.w, slots = g.kh * cut.line;
        for (int o = wave * 64; o < (slots << cut.lg_pieces); o += kRegThreads) {
            const int i = o + lane, q = i >> cut.lg_pieces, c = (i ^ (q >> 1)) & (pieces - 1);
            const int k = (int)fast_div((uint32_t)q, cut.by_line), t = q - k * cut.line;
            const int pix = first + (k * g.dh - g.ph) * g.w - g.pw + t, ch = win0 + c * 8;
            const bool ok = q < slots && pix >= 0 && pix < npix && ch < g.c_in;
            dma_load16(rsrc_x, ok ? (uint32_t)(pix * g.c_in + ch) * 2u : kOutOfRange,
                       __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)o * 16u));
        }
        // ---- taps in use: this wave's share of them, for all positions ----
        const bool packed = (g.flags & FC_PACKED_MASKS) != 0;
        const int pp = kept ? p : 0;
        const int r = (int)fast_div((uint32_t)pp, g.div_wo), ow = pp - r * g.wo;
        const int img = (int)fast_div((uint32_t)r, g.div_ho), oh = r - img * g.ho;
        __syncthreads(); // bits_s cleared
        uint32_t mine = 0;
        constexpr int U = 3; // look-ups in flight
        for (int t0 = wave; t0 < taps; t0 += 4 * U) {
            bool in[U];
            uint8_t m[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int t = t0 + 4 * u, kh = (int)fast_div((uint32_t)t, cut.by_kw), kw = t - kh * g.kw;
                const int ih = oh - g.ph + kh * g.dh, iw = ow - g.pw + kw * g.dw;
                in[u] = kept && t < taps && (uint32_t)ih < (uint32_t)g.h && (uint32_t)iw < (uint32_t)g.w;
                m[u] = mask_in ? (uint8_t)mask_at(mask_in, in[u] ? (img * g.h + ih) * g.w + iw : 0, packed) : (uint8_t)1;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) mine |= in[u] && m[u] ? 1u << (t0 + 4 * u) : 0u;
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
    if (co0 >= g.c_out || n == 0) return;

    // ---- this wave's 16 channels: weights from LDS to registers, and where their pieces lie ----
    const int ic = cog >= 16 ? cig : (16 / cog) * cig, ppt = ic >> 3;
    const int bw0 = (co0 / cog) * cig;             // first input channel of the block's groups
    const int co = co0 + col, wch = (co / cog) * cig;
    u32x4_t wf[KS];
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
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
            const int local = bw0 + pc * 8 + hf * 4 - wch;
            const bool ok = tap < taps && local >= 0 && local < cig;
            const uint2 v = ok ? *reinterpret_cast<const uint2 *>(w_s + (((co - blk0) * taps + tap) * cig + local) * 2) : make_uint2(0, 0);
            wf[s][2 * hf] = v.x;
            wf[s][2 * hf + 1] = v.y;
        }
    }
    float4 bq = make_float4(0.f, 0.f, 0.f, 0.f);
    if (bias) bq = *reinterpret_cast<const float4 *>(bias + co0 + quarter * 4);
    const uint32_t zero_at = (uint32_t)(cut.x_bytes + cut.w_bytes), pmask = (1u << cut.lg_pieces) - 1u;
    for (int r0 = 0; r0 < n; r0 += 16) {
        const bool live = r0 + col < n;
        const int j = live ? order_s[r0 + col] : 0;
        const uint32_t bits = live ? bits_s[j] : 0u;
        u32x4_t xv[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const uint32_t q = (uint32_t)(j + xq[s]);
            const uint32_t at = ((q << cut.lg_pieces) + ((xc[s] ^ (q >> 1)) & pmask)) * 16u;
            xv[s] = *reinterpret_cast<const u32x4_t *>(lds + ((bits & xsel[s]) ? at : zero_at));
        }
        f32x4_t acc = {bq.x, bq.y, bq.z, bq.w};
#pragma unroll
        for (int s = 0; s < KS; ++s) acc = mfma16<DT>(wf[s], xv[s], acc);
        if (g.flags & FC_RELU)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] = !(acc[i] > 0.f) ? (acc[i] != acc[i] ? acc[i] : 0.f) : acc[i];
        if (live)
            store4<DT, TO>(out + (int64_t)(first + j) * g.c_out + co0 + quarter * 4, acc[0], acc[1], acc[2], acc[3]);
    }
}

// matrix steps of a 16-channel block's reduction
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
    // whole 16-channel blocks that do not cut a group boundary; windows of whole 16-byte pieces
    if (g.c_out % 16 != 0 || g.c_in % 8 != 0 || cig % 4 != 0) return false;
    if (cog < 16 ? 16 % cog != 0 : cog % 16 != 0) return false;
    if ((cog >= 16 ? cig : (16 / cog) * cig) % 8 != 0) return false;
    if (g.kh * g.kw > 32 || grouped_steps(g, cig, cog) > 18) return false; // tap bits; weights in registers
    if (g.h > 16384 || g.w > 16384 || g.ph > 8192 || g.pw > 8192) return false;
    return (uint64_t)g.n * g.h * g.w * g.c_in * 2u < kBufferLimit && (uint64_t)g.c_out * g.kh * g.kw * cig * 2u < kBufferLimit;
}

template <int DT, typename TO>
static hipError_t launch_grouped(const Geom &g, int groups, const void *x, const uint8_t *mask_in, const uint8_t *mask_out,
                                 const void *w, const float *bias, const int32_t *idx, const int32_t *count, void *out,
                                 hipStream_t s)
{
    const int cig = g.c_in / groups, cog = g.c_out / groups;
    // spans of positions as windows of pixels: unit stride, same size, no list, groups that do not straddle a
    // workgroup's 64 channels and whose channels make a power of two of 16-byte pieces, at most 64 KB of LDS
    const int wch = cog <= 64 && 64 % cog == 0 ? 64 / cog * cig : 0;
    if (!idx && g.sh == 1 && g.sw == 1 && g.ho == g.h && g.wo == g.w && wch >= 32 && wch <= 128 && (wch & (wch - 1)) == 0 &&
        grouped_steps(g, cig, cog) <= 9) {
        WindowCut cut;
        cut.line = kWindowSpan + (g.kw - 1) * g.dw;
        cut.lg_pieces = wch == 32 ? 2 : (wch == 64 ? 3 : 4);
        cut.x_bytes = (g.kh * cut.line * wch * 2 + 1023) & ~1023;
        cut.w_bytes = (64 * g.kh * g.kw * cig * 2 + 1023) & ~1023;
        cut.by_line = make_fastdiv((uint32_t)cut.line);
        cut.by_kw = make_fastdiv((uint32_t)g.kw);
        cut.by_ppt = make_fastdiv((uint32_t)((cog >= 16 ? cig : (16 / cog) * cig) / 8));
        const int bytes = cut.x_bytes + cut.w_bytes + 16 + kWindowSpan * 5;
        if (bytes <= 64 * 1024) {
            auto kern = grouped_steps(g, cig, cog) <= 5 ? k_conv_grouped_window<DT, TO, 5> : k_conv_grouped_window<DT, TO, 9>;
            hipLaunchKernelGGL(kern, dim3((g.m + kWindowSpan - 1) / kWindowSpan, (g.c_out + 63) / 64), dim3(kRegThreads), bytes, s,
                               g, cut, cig, cog, (const uint16_t *)x, mask_in, mask_out, (const uint16_t *)w, bias, (TO *)out);
            return hipGetLastError();
        }
    }
    const dim3 grid((g.m + kGroupedSpan - 1) / kGroupedSpan, (g.c_out + 63) / 64);
    const int steps = grouped_steps(g, cig, cog);
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
