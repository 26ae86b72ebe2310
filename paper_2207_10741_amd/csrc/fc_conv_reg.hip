// Focused convolution whose matrix operands go straight from global memory into registers:
// fp32 storage (any channel counts) and grouped layers of 16-bit storage.
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
    for (int i = tid; i < n * taps; i += kRegThreads) {
        const int r = (int)((uint32_t)i / (uint32_t)taps), t = i - r * taps;
        const int kh = (int)((uint32_t)t / (uint32_t)g.kw), kw = t - kh * g.kw;
        const int ih = (int)(int16_t)(s.hw[r] & 0xffff) + kh * g.dh, iw = (s.hw[r] >> 16) + kw * g.dw;
        bool ok = ih >= 0 && ih < g.h && iw >= 0 && iw < g.w;
        if (ok && mask_in) ok = mask_at(mask_in, (int64_t)(s.img[r] * g.h + ih) * g.w + iw, packed);
        if (ok) atomicOr(&s.bits[t >> 5][r], 1u << (t & 31));
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
// A wave owns 32 rows x NB * 32 output channels.  One step = 16 input channels of one tap: lane
// (row, half) holds channels 4 * half .. + 3 of each 8-channel piece of its row as one 16-byte load,
// and the four elements feed four matrix instructions whose reduction pair is (element e of the
// lower half, element e of the upper half); both operands are loaded the same way, so the
// pairing of channels is the same.  Three register sets: the loads of step s + 2 are issued before
// step s is multiplied.
//
// KSPLIT: the four waves of a workgroup take the same 32 rows and a quarter of the reduction
// each and add up in LDS, in wave order: a layer of a few hundred row blocks is then spread over
// four times as many SIMDs (64 -> 64 on 2 x 60 x 80 positions, 48 % irrelevant: 66 us on
// the vector ALUs with 5 us each of compaction and zero-fill).  Otherwise the waves take 32 rows
// each of a 128-position span.
// ---------------------------------------------------------------------------------------------
template <int NB, bool KSPLIT>
__global__ __launch_bounds__(kRegThreads, 2) void k_conv_f32(Geom g, const float *__restrict__ x,
                                                             const uint8_t *__restrict__ mask_in,
                                                             const uint8_t *__restrict__ mask_out,
                                                             const float *__restrict__ w,
                                                             const float *__restrict__ bias,
                                                             const int32_t *__restrict__ idx,
                                                             const int32_t *__restrict__ count, float *__restrict__ out)
{
    constexpr int S = KSPLIT ? 32 : 128;
    constexpr int NQ = NB * 4; // accumulator quads (4 channels of one position) per lane
    __shared__ SpanRows rows_s;
    __shared__ float4 part[KSPLIT ? 4 * NQ * 64 : 1];
    const int rows = idx ? *count : g.m;
    const int first = blockIdx.x * S;
    if (first >= rows) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5, l32 = lane & 31;
    const int co0 = blockIdx.y * (NB * 32);
    int n, nd;
    span_rows<S>(g, mask_in, mask_out, idx, rows, first, rows_s, &n, &nd);
    if (nd && !(g.flags & FC_SKIP_ZERO_FILL))
        clear_dropped<float>(rows_s, nd, out, g.c_out, co0, min(NB * 32, g.c_out - co0));
    const int r0 = KSPLIT ? 0 : wave * 32;
    if (r0 >= n) return; // (KSPLIT: the whole workgroup; otherwise nothing below waits for this wave)

    const int taps = g.kh * g.kw;
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(x), 0, (uint32_t)g.n * g.h * g.w * g.c_in * 4u, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(w), 0, (uint32_t)g.c_out * taps * g.c_in * 4u, 0x00020000);
    const int r = r0 + l32;
    const bool live = r < n;
    const uint32_t xbase = live ? (uint32_t)(rows_s.base[r] * g.c_in + half * 4) * 4u : 0u;
    const uint64_t bits = live ? (rows_s.bits[0][r] | ((uint64_t)rows_s.bits[1][r] << 32)) : 0ull;
    uint32_t wbase[NB];
    bool wlive[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int co = co0 + b * 32 + l32;
        wlive[b] = co < g.c_out;
        wbase[b] = (uint32_t)(co * taps * g.c_in + half * 4) * 4u;
    }

    const int cch = (g.c_in + 15) >> 4, steps = taps * cch;
    const int s0 = KSPLIT ? wave * steps / 4 : 0, s1 = KSPLIT ? (wave + 1) * steps / 4 : steps;
    const bool by4 = (g.c_in & 3) == 0;
    const int tail = g.c_in - (cch - 1) * 16; // channels of a tap's last step (1 .. 16)
    // cursor of the next step to load
    int tap = s0 / cch, cc = s0 - tap * cch, kh = tap / g.kw, kw = tap - kh * g.kw;

    f32x16_t acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[b][i] = 0.f;

    u32x4_t xv[3][2], wv[3][NB][2];
    auto load = [&](auto set_c) __attribute__((always_inline)) {
        constexpr int st = decltype(set_c)::value;
        const uint32_t sx = (uint32_t)((kh * g.dh * g.w + kw * g.dw) * g.c_in + cc * 16) * 4u;
        const uint32_t sw = (uint32_t)(tap * g.c_in + cc * 16) * 4u;
        const bool tap_ok = (bits >> tap) & 1u;
        const int left = g.c_in - cc * 16 - half * 4; // channels from this lane's first one to the end
        if (by4 || cc + 1 < cch) {
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const bool in = p * 8 < left;
                xv[st][p] = __builtin_amdgcn_raw_buffer_load_b128(rx, tap_ok && in ? xbase + sx + p * 32u : kOutOfRange, 0, 0);
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    wv[st][b][p] = __builtin_amdgcn_raw_buffer_load_b128(
                        rw, wlive[b] && in ? wbase[b] + sw + p * 32u : kOutOfRange, 0, 0);
            }
        } else {
            // the last channels of a row whose length is no multiple of four: one by one
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool in = p * 8 + e < left;
                    const uint32_t o = p * 32u + e * 4u;
                    xv[st][p][e] = __builtin_amdgcn_raw_buffer_load_b32(rx, tap_ok && in ? xbase + sx + o : kOutOfRange, 0, 0);
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        wv[st][b][p][e] =
                            __builtin_amdgcn_raw_buffer_load_b32(rw, wlive[b] && in ? wbase[b] + sw + o : kOutOfRange, 0, 0);
                }
        }
        if (++cc == cch) {
            cc = 0;
            ++tap;
            if (++kw == g.kw) {
                kw = 0;
                ++kh;
            }
        }
    };
    int mcc = cc; // channel step of the next step to multiply
    auto multiply = [&](auto set_c) __attribute__((always_inline)) {
        constexpr int st = decltype(set_c)::value;
        __builtin_amdgcn_sched_barrier(0);
        const bool whole = mcc + 1 < cch || tail > 8; // (otherwise the upper eight channels do not exist)
        mcc = mcc + 1 == cch ? 0 : mcc + 1;
#pragma unroll
        for (int p = 0; p < 2; ++p)
            if (p == 0 || whole)
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(wv[st][b][p][e]),
                                                                      __uint_as_float(xv[st][p][e]), acc[b], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    using C0 = std::integral_constant<int, 0>;
    using C1 = std::integral_constant<int, 1>;
    using C2 = std::integral_constant<int, 2>;
    if (s0 < s1) load(C0{});
    if (s0 + 1 < s1) load(C1{});
    for (int s = s0; s < s1; s += 3) {
        if (s + 2 < s1) load(C2{});
        multiply(C0{});
        if (s + 1 >= s1) break;
        if (s + 3 < s1) load(C0{});
        multiply(C1{});
        if (s + 2 >= s1) break;
        if (s + 4 < s1) load(C1{});
        multiply(C2{});
    }

    // a lane's quad (b, q) = channels co0 + 32 b + 8 q + 4 half .. + 3 of position p
    auto finish = [&](int b, int q, float4 v) __attribute__((always_inline)) {
        const int co = co0 + b * 32 + q * 8 + half * 4;
        float e[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (bias && co + i < g.c_out) e[i] += bias[co + i];
            if (g.flags & FC_RELU) e[i] = !(e[i] > 0.f) ? (e[i] != e[i] ? e[i] : 0.f) : e[i];
        }
        if (!live) return;
        float *o = out + (int64_t)rows_s.p[r] * g.c_out + co;
        if ((g.c_out & 3) == 0) {
            if (co < g.c_out) *reinterpret_cast<float4 *>(o) = make_float4(e[0], e[1], e[2], e[3]);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (co + i < g.c_out) o[i] = e[i];
        }
    };
    if constexpr (KSPLIT) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                part[(wave * NQ + b * 4 + q) * 64 + lane] =
                    make_float4(acc[b][q * 4], acc[b][q * 4 + 1], acc[b][q * 4 + 2], acc[b][q * 4 + 3]);
        __syncthreads();
        // wave v finishes quad v of every 32-channel block
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            float4 v = part[(b * 4 + wave) * 64 + lane];
#pragma unroll
            for (int k = 1; k < 4; ++k) {
                const float4 t = part[(k * NQ + b * 4 + wave) * 64 + lane];
                v.x += t.x; v.y += t.y; v.z += t.z; v.w += t.w;
            }
            finish(b, wave, v);
        }
    } else {
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                finish(b, q, make_float4(acc[b][q * 4], acc[b][q * 4 + 1], acc[b][q * 4 + 2], acc[b][q * 4 + 3]));
    }
}

// 64 taps: the tap-valid bits of a row; 32-bit byte offsets into x and w; row origins in 16 bits
bool conv_f32_supported(const Geom &g)
{
    return g.kh * g.kw <= 64 && g.h <= 16384 && g.w <= 16384 && g.ph <= 8192 && g.pw <= 8192 &&
           (uint64_t)g.n * g.h * g.w * g.c_in * 4u < kBufferLimit &&
           (uint64_t)g.c_out * g.kh * g.kw * g.c_in * 4u < kBufferLimit;
}

template <int NB, bool KSPLIT>
static hipError_t launch_f32(const Geom &g, const void *x, const uint8_t *mask_in, const uint8_t *mask_out, const void *w,
                             const float *bias, const int32_t *idx, const int32_t *count, void *out, hipStream_t s)
{
    constexpr int S = KSPLIT ? 32 : 128;
    hipLaunchKernelGGL((k_conv_f32<NB, KSPLIT>), dim3((g.m + S - 1) / S, (g.c_out + NB * 32 - 1) / (NB * 32)),
                       dim3(kRegThreads), 0, s, g, (const float *)x, mask_in, mask_out, (const float *)w, bias, idx, count,
                       (float *)out);
    return hipGetLastError();
}

hipError_t launch_conv_f32(const Geom &g, const void *x, const uint8_t *mask_in, const uint8_t *mask_out, const void *w,
                           const float *bias, const int32_t *idx, const int32_t *count, void *out, hipStream_t s)
{
    // 64 output channels per wave halve the reading of x; an odd number of 32-channel blocks would
    // leave half of the last pair idle
    const int blocks32 = (g.c_out + 31) / 32;
    const bool wide = blocks32 % 2 == 0;
    // one wave per 32 rows would give fewer than one wave per SIMD: split the reduction
    const int64_t waves = (int64_t)((g.m + 31) / 32) * (wide ? blocks32 / 2 : blocks32);
    const bool ksplit = waves < 1024;
    if (wide)
        return ksplit ? launch_f32<2, true>(g, x, mask_in, mask_out, w, bias, idx, count, out, s)
                      : launch_f32<2, false>(g, x, mask_in, mask_out, w, bias, idx, count, out, s);
    return ksplit ? launch_f32<1, true>(g, x, mask_in, mask_out, w, bias, idx, count, out, s)
                  : launch_f32<1, false>(g, x, mask_in, mask_out, w, bias, idx, count, out, s);
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
    constexpr int S = kMaxSpan;
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
        const bool live = r < n;
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
    if (n > 0) load(C0{}, col);
    for (int r = col; r - col < n; r += 32) {
        if (r - col + 16 < n) load(C1{}, r + 16);
        multiply(C0{}, r);
        if (r - col + 16 >= n) break;
        if (r - col + 32 < n) load(C0{}, r + 32);
        multiply(C1{}, r + 16);
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
    const dim3 grid((g.m + kMaxSpan - 1) / kMaxSpan, (g.c_out + 63) / 64);
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
