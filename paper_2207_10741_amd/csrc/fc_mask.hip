// Mask-side kernels: mask propagation (Sec. III-B), ordered compaction of the kept
// positions (Sec. III-A: which patches become columns) fused with it, zero-fill of
// the irrelevant output rows for the direct-convolution path, and the max-pool
// helper.  All of them are byte/row movers bound by HBM bandwidth or launch latency.
#include "fc_internal.hpp"

namespace fc {

// ---------------------------------------------------------------------------
// Mask propagation: one thread per output byte; the byte under the centre tap.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_mask_downsample(const uint8_t *__restrict__ mask_in, int n, int h,
                                                         int w, int ch0, int cw0, int sh, int sw, int ho,
                                                         int wo, uint8_t *__restrict__ mask_out)
{
    const int64_t total = (int64_t)n * ho * wo;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < total;
         p += (int64_t)gridDim.x * blockDim.x) {
        // (position counts fit 31 bits: 32-bit divisions)
        const uint32_t t = (uint32_t)p / (uint32_t)wo;
        const int ow = (int)((uint32_t)p - t * (uint32_t)wo);
        const int b = (int)(t / (uint32_t)ho);
        const int oh = (int)(t - (uint32_t)b * (uint32_t)ho);
        int ih = min(max(oh * sh + ch0, 0), h - 1);
        int iw = min(max(ow * sw + cw0, 0), w - 1);
        mask_out[p] = mask_in[(b * h + ih) * w + iw] ? 1 : 0;
    }
}

hipError_t launch_mask_downsample(const uint8_t *mask_in, int n, int h, int w, int kh, int kw, int sh,
                                  int sw, int ph, int pw, int dh, int dw, int ho, int wo,
                                  uint8_t *mask_out, hipStream_t s)
{
    const int64_t total = (int64_t)n * ho * wo;
    int blocks = (int)((total + 255) / 256);
    if (blocks > 65536) blocks = 65536;
    const int ch0 = -ph + dh * ((kh - 1) / 2), cw0 = -pw + dw * ((kw - 1) / 2);
    hipLaunchKernelGGL(k_mask_downsample, dim3(blocks), dim3(256), 0, s, mask_in, n, h, w, ch0, cw0, sh, sw,
                       ho, wo, mask_out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Patch labels by a window rule (the other readings of "a patch labelled irrelevant",
// Sec. III-A): kept if ANY pixel of the window is relevant, or only if ALL are.  Pixels
// outside the image are not part of the window.  One thread per output byte; the
// window's mask bytes come through the cache (neighbouring positions share them).
// ---------------------------------------------------------------------------
template <bool ALL>
__global__ __launch_bounds__(256) void k_mask_window(const uint8_t *__restrict__ mask_in, int n, int h, int w,
                                                     int kh, int kw, int sh, int sw, int ph, int pw, int dh,
                                                     int dw, int ho, int wo, uint8_t *__restrict__ mask_out)
{
    const int64_t total = (int64_t)n * ho * wo;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < total;
         p += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t t = (uint32_t)p / (uint32_t)wo; // (position counts fit 31 bits)
        const int ow = (int)((uint32_t)p - t * (uint32_t)wo);
        const uint32_t b = t / (uint32_t)ho;
        const int oh = (int)(t - b * (uint32_t)ho);
        const uint8_t *img = mask_in + (int64_t)b * ((int64_t)h * w);
        int inside = 0, relevant = 0;
        for (int i = 0; i < kh; ++i) {
            const int ih = oh * sh - ph + i * dh;
            if (ih < 0 || ih >= h) continue;
            for (int j = 0; j < kw; ++j) {
                const int iw = ow * sw - pw + j * dw;
                if (iw < 0 || iw >= w) continue;
                ++inside;
                relevant += img[(int64_t)ih * w + iw] != 0;
            }
        }
        mask_out[p] = ALL ? (inside > 0 && relevant == inside) : (relevant > 0);
    }
}

hipError_t launch_mask_window(const uint8_t *mask_in, int n, int h, int w, int kh, int kw, int sh, int sw,
                              int ph, int pw, int dh, int dw, int ho, int wo, bool all, uint8_t *mask_out,
                              hipStream_t s)
{
    const int64_t total = (int64_t)n * ho * wo;
    int blocks = (int)((total + 255) / 256);
    if (blocks > 65536) blocks = 65536;
    if (all)
        hipLaunchKernelGGL(k_mask_window<true>, dim3(blocks), dim3(256), 0, s, mask_in, n, h, w, kh, kw, sh, sw, ph,
                           pw, dh, dw, ho, wo, mask_out);
    else
        hipLaunchKernelGGL(k_mask_window<false>, dim3(blocks), dim3(256), 0, s, mask_in, n, h, w, kh, kw, sh, sw, ph,
                           pw, dh, dw, ho, wo, mask_out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Ordered kept lists (Sec. III-A: which patches become columns) fused with the mask
// propagation (Sec. III-B), for one mask or for all levels of a pyramid.  A workgroup owns 4096
// consecutive positions of one list, a lane PER of them: it labels them in the
// input mask (one load for a list at the mask's own resolution, PER byte loads in flight
// otherwise), ranks them by a prefix sum (vector ALU inside a wave, LDS across the
// waves) and stores the kept ones.  PER = 4 (1024 threads) for the latency of short lists, 16 (256 threads) for the
// throughput of long ones, see launch_lists_n.  Bound: launch latency for the masks of one image, HBM for the
// largest.  No workgroup ever waits on another, so every grid drains:
//   - short lists: ONE launch; a workgroup counts the kept positions before its own by itself (16 bytes per
//     lane and load, also through a stride);
//   - longer lists: two launches, labels and per-workgroup counts first, then offsets and lists.
// (Four levels of one 224 x 224 mask: 7.1 + 4.2 us in two launches with sixteen positions per lane and the
// levels' maps applied one after another; the labels of 5 814 positions through a stride: 8.9 us.)
// ---------------------------------------------------------------------------
constexpr int kListThreads = 1024; // of a workgroup whose lanes take four positions
constexpr int kListWaves = kListThreads / 64;
template <int PER> constexpr int kThreadsOf = kCompactBlockElems / PER;
// 16-byte reads of a list's last workgroup (off their alignment they count twice) up to which one launch serves all lists, and up to which its workgroups have 256 threads
// (kOnceBlocks: where a list has to be labelled position by position).  One launch after another, bytes, us, two launches -> here: four levels of 160 x 160
// (1 600 reads) 6.1 -> 3.6, 224 x 224 (3 136) 6.2 -> 4.4, 251 x 333 (5 224) 6.4 -> 5.5, 2 x 224 x 224 (6 272) 6.4 -> 5.4, 8 x 131 x 127 (8 320) 6.4 -> 5.3, 12 x 128 x 128
// (12 288) 6.8 -> 6.7, 4 x 224 x 224 (12 544) 6.6 -> 7.0, 16 x 128 x 128 (16 384) 7.3 -> 6.8; one list of the last two 5.9 -> 4.8 and 5.9 -> 5.3.  With 256 threads 2 x 224 x 224, 8 x 131
// x 127, 4 x 224 x 224 and 16 x 128 x 128 take 5.7, 6.0, 8.1 and 9.2; with 1024 160 x 160 and 224 x 224 take 4.4 and 5.2.  Past 16 384 the counting alone is what the
// second launch costs.
// Through a stride less: a list and the layer behind it, two launches -> one: 12 x 112 x 112 / 2 (4 704 reads) 11.7 -> 10.8, 10 x 130 x 130 / 2 (11 700)
// 12.2 -> 13.6, 14 x 105 x 131 / 2 (13 356) 12.2 -> 14.0.
constexpr int kOncePieces = 16384, kOncePiecesStepped = 10000, kBriefPieces = 4096, kOnceBlocks = 4;
// Workgroups of a list at the mask's resolution from which on a lane takes sixteen positions: there the labels of
// sixteen are one load as those of four are, and what such a list costs is instructions per lane.  Four -> sixteen, a list
// alone / a pyramid of four levels: 1.6 M positions 10.1 -> 9.9 / 12.4 -> 12.4 us, 2.1 M 10.1 -> 10.0 / 13.9 -> 12.8, 5.2 M
// 14.6 -> 11.4 / 23.1 -> 18.3, 16.6 M 34.5 -> 20.9 / 57.2 -> 42.0.  (Below the line, or where the first level has a stride,
// four stay ahead: 0.8 M 10.2 against 11.4 us, three strided levels of 16.6 M 22.0 against 23.3.)
constexpr int kLongBlocks = 400;

// sum of v over the workgroup (all threads get it)
template <int WAVES>
__device__ __forceinline__ int block_sum(int v, int *scratch)
{
    const int incl = wave_inclusive_scan(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 63) scratch[threadIdx.x >> 6] = incl;
    __syncthreads();
    int s = 0;
#pragma unroll
    for (int i = 0; i < WAVES; ++i) s += scratch[i];
    return s;
}

// 0x80 in every nonzero byte
__device__ __forceinline__ uint32_t nonzero_bytes(uint32_t v) { return (((v & 0x7f7f7f7fu) + 0x7f7f7f7fu) | v) & 0x80808080u; }

// bit j = position p0 + j of the list is kept, j < PER (p0 a multiple of PER; positions past the end read as 0)
template <int PER>
__device__ __forceinline__ uint32_t labels(const LabelMap &L, const uint8_t *__restrict__ mask_in, int p0, bool vec)
{
    if (p0 >= L.m) return 0;
    const int left = L.m - p0;
    if (L.identity && L.packed_in) {
        const uint32_t f = (reinterpret_cast<const uint32_t *>(mask_in)[p0 >> 5] >> (p0 & 31)) & ((1u << PER) - 1u);
        return left < PER ? f & ((1u << left) - 1u) : f;
    }
    if (L.identity && vec && left >= PER) {
        auto four = [](uint32_t w) {
            const uint32_t v = nonzero_bytes(w);
            return ((v >> 7) & 1u) | ((v >> 14) & 2u) | ((v >> 21) & 4u) | (v >> 28);
        };
        if constexpr (PER == 4) {
            return four(*reinterpret_cast<const uint32_t *>(mask_in + p0));
        } else {
            const uint4 v = *reinterpret_cast<const uint4 *>(mask_in + p0);
            return four(v.x) | (four(v.y) << 4) | (four(v.z) << 8) | (four(v.w) << 12);
        }
    }
    const uint32_t t = fast_div((uint32_t)p0, L.div_w);
    int ow = p0 - (int)t * L.wl;
    int b = (int)fast_div(t, L.div_h), oh = (int)t - b * L.hl;
    auto along = [](const AxisMap &a, int v) { return min(max(v * a.mul + a.add, a.lo), a.hi); };
    int row_at = (b * L.h0 + along(L.row, oh)) * L.w0;
    int at[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        at[j] = j < left ? row_at + along(L.col, ow) : -1;
        if (++ow == L.wl) {
            ow = 0;
            if (++oh == L.hl) {
                oh = 0;
                ++b;
            }
            row_at = (b * L.h0 + along(L.row, oh)) * L.w0;
        }
    }
    uint32_t f = 0;
    if (L.packed_in) {
        uint32_t got[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) got[j] = at[j] >= 0 ? reinterpret_cast<const uint32_t *>(mask_in)[at[j] >> 5] : 0u;
#pragma unroll
        for (int j = 0; j < PER; ++j) f |= ((got[j] >> (at[j] & 31)) & 1u) << j;
    } else {
        uint8_t got[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) got[j] = at[j] >= 0 ? mask_in[at[j]] : (uint8_t)0;
#pragma unroll
        for (int j = 0; j < PER; ++j) f |= got[j] ? 1u << j : 0u;
    }
    return f;
}

// Labels of positions p0 .. p0 + PER - 1 to mask_out (bytes 0 / 1, or bits, zeros up to a whole 64-bit word).
// All lanes call it.
template <int PER>
__device__ __forceinline__ void store_labels(const LabelMap &L, int p0, uint32_t f)
{
    if (!L.mask_out) return;
    if (L.packed_out) {
        const int lane = threadIdx.x & 63;
        uint32_t v = f;
        if constexpr (PER == 4) { // four lanes make a 16-bit piece
            v <<= 4 * (lane & 3);
            v |= __shfl_xor(v, 1);
            v |= __shfl_xor(v, 2);
        }
        if ((PER == 16 || (lane & 3) == 0) && (int64_t)p0 < (((int64_t)L.m + 63) & ~(int64_t)63)) reinterpret_cast<uint16_t *>(L.mask_out)[p0 >> 4] = (uint16_t)v;
        return;
    }
    if (p0 + PER <= L.m) {
        auto bytes = [](uint32_t v) { return (v & 1u) | ((v & 2u) << 7) | ((v & 4u) << 14) | ((v & 8u) << 21); };
        if constexpr (PER == 4)
            *reinterpret_cast<uint32_t *>(L.mask_out + p0) = bytes(f);
        else
            *reinterpret_cast<uint4 *>(L.mask_out + p0) = make_uint4(bytes(f), bytes(f >> 4), bytes(f >> 8), bytes(f >> 12));
    } else {
        for (int j = 0; j < PER && p0 + j < L.m; ++j) L.mask_out[p0 + j] = (f >> j) & 1u;
    }
}

template <int NL>
__device__ __forceinline__ int list_of_block(const ListArgs<NL> &a, int block)
{
    int l = 0;
#pragma unroll
    for (int i = 1; i < NL; ++i)
        if (i < a.lists && block >= a.at[i].block0) l = i;
    return l;
}

// the workgroup's part of the list: kept positions p0 .. p0 + PER - 1 of every lane after `base` earlier ones;
// returns the number kept by the whole workgroup.  `staged`: the list is put together in LDS and leaves in
// whole lines (long lists: 8.3 million entries 38 us straight from the lanes)
template <int PER>
__device__ __forceinline__ int store_list(const LabelMap &L, int p0, uint32_t f, int base, int *wave_sum,
                                          int32_t *staged = nullptr)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = __popc(f), incl = wave_inclusive_scan(c);
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    int before = 0, total = 0;
#pragma unroll
    for (int i = 0; i < kThreadsOf<PER> / 64; ++i) {
        const int t = wave_sum[i];
        before += i < wave ? t : 0;
        total += t;
    }
    int32_t *to = (staged ? staged : L.idx + base) + (before + incl - c);
    if constexpr (PER == 4) {
#pragma unroll
        for (int j = 0; j < PER; ++j)
            if ((f >> j) & 1u) *to++ = p0 + j;
    } else {
        for (; f; f &= f - 1) *to++ = p0 + __ffs((int)f) - 1;
    }
    if (staged) {
        __syncthreads();
        for (int i = threadIdx.x; i < total; i += kThreadsOf<PER>) L.idx[(int64_t)base + i] = staged[i];
    }
    return total;
}

// sum + nonzero bytes of v (the masked byte differences of v ^ 1 and v: one for every byte that is not zero)
__device__ __forceinline__ uint32_t add_nonzero(uint32_t v, uint32_t sum) { return __builtin_amdgcn_msad_u8(v ^ 0x01010101u, v, sum); }

// How a list steps through a byte mask, for the one-launch form.  pieces: 16-byte pieces of a row that hold its positions' bytes, 0 where positions
// are not `col.mul` bytes apart (a divisor of 16), per: positions of a piece, sel: their bytes in words 0, 1 and 3, 2 of a piece
struct RowPieces {
    int32_t pieces, per, rows_in; // rows_in: rows of the whole input mask
    uint32_t sel, sel_odd, sel_rest;
    FastDiv div_pieces;
};
template <int NL> struct RowPiecesArgs {
    RowPieces at[NL];
};

// Kept positions among the first `before` of a list, this lane's share of them (the workgroup's lanes share all): 16 bytes a load, B loads in
// flight.  A row of a list that steps through the mask is read by pieces that start at its first position's byte.
template <int THREADS, int B>
__device__ __forceinline__ int kept_before(const LabelMap &L, const RowPieces &P, const uint8_t *__restrict__ mask_in, int before)
{
    uint32_t part = 0;
    if (L.identity) {
        const uint4 *m4 = reinterpret_cast<const uint4 *>(mask_in);
        const int pieces = before >> 4; // (a multiple of 16)
        for (int i0 = threadIdx.x; i0 < pieces; i0 += B * THREADS) {
            uint4 v[B];
#pragma unroll
            for (int k = 0; k < B; ++k) v[k] = i0 + k * THREADS < pieces ? m4[i0 + k * THREADS] : make_uint4(0, 0, 0, 0);
#pragma unroll
            for (int k = 0; k < B; ++k) part = add_nonzero(v[k].w, add_nonzero(v[k].z, add_nonzero(v[k].y, add_nonzero(v[k].x, part))));
        }
        return part;
    }
    const int full = (int)fast_div((uint32_t)before, L.div_w), rest = before - full * L.wl; // whole rows, positions of the next
    const int pieces = full * P.pieces + (rest ? P.pieces : 0), bytes = P.rows_in * L.w0;
    for (int i0 = threadIdx.x; i0 < pieces; i0 += B * THREADS) {
        uint4 v[B];
        int n[B]; // positions of the piece that count
#pragma unroll
        for (int k = 0; k < B; ++k) {
            const int i = i0 + k * THREADS;
            const int r = (int)fast_div((uint32_t)i, P.div_pieces), q = i - r * P.pieces;
            const int b = (int)fast_div((uint32_t)r, L.div_h), oh = r - b * L.hl;
            n[k] = i < pieces ? min((r < full ? L.wl : rest) - q * P.per, P.per) : 0;
            const int ih = min(max(oh * L.row.mul + L.row.add, L.row.lo), L.row.hi);
            const int at = (b * L.h0 + ih) * L.w0 + L.col.add + q * 16;
            v[k] = make_uint4(0, 0, 0, 0);
            if (n[k] > 0) {
                if (at <= bytes - 16) { // (the sum could pass 31 bits)
                    __builtin_memcpy(&v[k], mask_in + at, 16);
                } else { // (the mask's last bytes)
                    for (int j = 0; j < n[k]; ++j) part += mask_in[at + j * L.col.mul] != 0;
                    n[k] = 0;
                }
            }
        }
#pragma unroll
        for (int k = 0; k < B; ++k) {
            uint32_t f[4] = {v[k].x & P.sel, v[k].y & P.sel_odd, v[k].z & P.sel_rest, v[k].w & P.sel_odd};
            const int end = n[k] * L.col.mul; // bytes of it
            if (n[k] < P.per)
#pragma unroll
                for (int j = 0; j < 4; ++j) f[j] &= end >= 4 * j + 4 ? ~0u : (end > 4 * j ? (1u << (8 * (end - 4 * j))) - 1u : 0u);
#pragma unroll
            for (int j = 0; j < 4; ++j) part = add_nonzero(f[j], part);
        }
    }
    return part;
}

// The labels of four positions of a list whose bytes are col.mul apart in a byte mask, at least four to a row.
__device__ __forceinline__ uint32_t labels_stepped(const LabelMap &L, const uint8_t *__restrict__ mask_in, int p0)
{
    if (p0 >= L.m) return 0;
    const int t = (int)fast_div((uint32_t)p0, L.div_w), ow = p0 - t * L.wl;
    auto row_at = [&](int r) {
        const int b = (int)fast_div((uint32_t)r, L.div_h), oh = r - b * L.hl;
        return (b * L.h0 + min(max(oh * L.row.mul + L.row.add, L.row.lo), L.row.hi)) * L.w0 + L.col.add;
    };
    const int here = L.wl - ow, left = L.m - p0; // positions to the end of the row, of the list
    const int at0 = row_at(t) + ow * L.col.mul, at1 = here < 4 && here < left ? row_at(t + 1) - here * L.col.mul : at0;
    uint32_t got[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) got[j] = j < left ? mask_in[(j < here ? at0 : at1) + j * L.col.mul] : 0u;
    return (got[0] ? 1u : 0u) | (got[1] ? 2u : 0u) | (got[2] ? 4u : 0u) | (got[3] ? 8u : 0u);
}

// One launch: labels, lists and counts.  A row of workgroups per list, four positions a lane; a workgroup counts the kept positions before
// its own by itself.  What this kernel takes is instructions, one wave's after another, and the round trip of the labels: 256 threads for
// the masks of an image, whose waves have a SIMD each, 1024 for longer ones, so that the last workgroups' counting
// has enough loads on its way.
template <int NL, int THREADS>
__global__ __launch_bounds__(THREADS) void k_lists_once(ListArgs<NL> a, RowPiecesArgs<NL> by_row, const uint8_t *__restrict__ mask_in)
{
    constexpr int W = THREADS / 64, ELEMS = THREADS * 4;
    __shared__ int wave_sum[2 * W];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const LabelMap &L = a.at[NL == 1 ? 0 : blockIdx.y];
    const RowPieces &P = by_row.at[NL == 1 ? 0 : blockIdx.y];
    const int before = blockIdx.x * ELEMS, p0 = before + tid * 4;
    if (before >= L.m) return;
    const bool vec = a.vec_in != 0;
    uint32_t f;
    int part = 0;
    if (L.identity ? vec && !L.packed_in : P.pieces > 0) {
        f = L.identity ? labels<4>(L, mask_in, p0, vec) : labels_stepped(L, mask_in, p0);
        part = kept_before<THREADS, 4>(L, P, mask_in, before);
    } else {
        f = labels<4>(L, mask_in, p0, vec);
        for (int b0 = 0; b0 < (int)blockIdx.x; b0 += 4) {
            uint32_t g[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) g[k] = b0 + k < (int)blockIdx.x ? labels<4>(L, mask_in, (b0 + k) * ELEMS + tid * 4, vec) : 0u;
#pragma unroll
            for (int k = 0; k < 4; ++k) part += __popc(g[k]);
        }
    }
    const int c = __popc(f), incl = wave_inclusive_scan(c), earlier = wave_inclusive_scan(part);
    if (lane == 63) {
        wave_sum[wave] = incl;
        wave_sum[W + wave] = earlier;
    }
    store_labels<4>(L, p0, f);
    __syncthreads();
    int at = incl - c, total = 0;
#pragma unroll
    for (int i = 0; i < W; ++i) {
        const int t = wave_sum[i], e = wave_sum[W + i];
        at += (i < wave ? t : 0) + e;
        total += t + e;
    }
    int32_t *to = L.idx + at;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if ((f >> j) & 1u) *to++ = p0 + j;
    if (tid == 0 && before + ELEMS >= L.m) *L.count = total;

    // on the side, for the convolution that follows: clear its split-K tile counters
    if (NL == 1 && a.ex.zero && blockIdx.x == 0)
        for (int i = tid; i < a.ex.zero_n; i += THREADS) a.ex.zero[i] = 0;
}

// two launches: labels and per-workgroup counts ...
template <int NL, int PER>
__global__ __launch_bounds__(kThreadsOf<PER>) void k_lists_count(ListArgs<NL> a, const uint8_t *__restrict__ mask_in,
                                                                 int32_t *__restrict__ block_counts)
{
    __shared__ int scratch[kThreadsOf<PER> / 64];
    const LabelMap &L = a.at[NL == 1 ? 0 : list_of_block(a, blockIdx.x)];
    const int p0 = (blockIdx.x - L.block0) * kCompactBlockElems + threadIdx.x * PER;
    const uint32_t f = labels<PER>(L, mask_in, p0, a.vec_in != 0);
    store_labels<PER>(L, p0, f);
    const int total = block_sum<kThreadsOf<PER> / 64>(__popc(f), scratch);
    if (threadIdx.x == 0) block_counts[blockIdx.x] = total;
}

// ... then offsets and lists (labels from mask_out where the first launch left them)
template <int NL, int PER>
__global__ __launch_bounds__(kThreadsOf<PER>) void k_lists_scatter(ListArgs<NL> a, const uint8_t *__restrict__ mask_in,
                                                                   const int32_t *__restrict__ block_counts)
{
    constexpr int W = kThreadsOf<PER> / 64;
    __shared__ int wave_sum[W], scratch[W];
    __shared__ int32_t staged[kCompactBlockElems];
    const int tid = threadIdx.x;
    const LabelMap &L = a.at[NL == 1 ? 0 : list_of_block(a, blockIdx.x)];
    const int p0 = (blockIdx.x - L.block0) * kCompactBlockElems + tid * PER;
    uint32_t f = 0;
    if (L.mask_out && p0 < L.m) {
        if (L.packed_out) {
            f = (reinterpret_cast<const uint32_t *>(L.mask_out)[p0 >> 5] >> (p0 & 31)) & ((1u << PER) - 1u); // (zeros past the end)
        } else if (p0 + PER <= L.m) {
            auto four = [](uint32_t v) { return (v & 1u) | ((v >> 7) & 2u) | ((v >> 14) & 4u) | ((v >> 21) & 8u); }; // bytes 0 / 1
            if constexpr (PER == 4) {
                f = four(*reinterpret_cast<const uint32_t *>(L.mask_out + p0));
            } else {
                const uint4 v = *reinterpret_cast<const uint4 *>(L.mask_out + p0);
                f = four(v.x) | (four(v.y) << 4) | (four(v.z) << 8) | (four(v.w) << 12);
            }
        } else {
            for (int j = 0; p0 + j < L.m; ++j) f |= L.mask_out[p0 + j] ? 1u << j : 0u;
        }
    } else if (!L.mask_out) {
        f = labels<PER>(L, mask_in, p0, a.vec_in != 0);
    }
    int part = 0;
    for (int i = L.block0 + tid; i < (int)blockIdx.x; i += kThreadsOf<PER>) part += block_counts[i];
    const int base = block_sum<kThreadsOf<PER> / 64>(part, scratch);
    const int total = store_list<PER>(L, p0, f, base, wave_sum, staged);
    if (tid == 0 && (int64_t)((int)blockIdx.x - L.block0 + 1) * kCompactBlockElems >= L.m) *L.count = base + total;
    if (NL == 1 && a.ex.zero && blockIdx.x == 0)
        for (int i = tid; i < a.ex.zero_n; i += kThreadsOf<PER>) a.ex.zero[i] = 0;
}

// Are the bytes of a list's positions col.mul apart along a row, so that 16-byte pieces hold 16 / col.mul of them each?
static RowPieces row_pieces(const LabelMap &L)
{
    RowPieces P = {};
    const int mul = L.col.mul;
    if (L.identity || L.packed_in || (mul != 1 && mul != 2 && mul != 4 && mul != 8 && mul != 16) || L.wl < 4 || L.col.add < 0) return P;
    if ((int64_t)(L.wl - 1) * mul + L.col.add > L.w0 - 1 || L.col.lo > L.col.add || L.col.hi < (L.wl - 1) * mul + L.col.add) return P;
    P.per = 16 / mul;
    P.pieces = (L.wl + P.per - 1) / P.per;
    P.div_pieces = make_fastdiv((uint32_t)P.pieces);
    P.rows_in = (int32_t)((int64_t)L.m / ((int64_t)L.hl * L.wl) * L.h0);
    P.sel = mul == 1 ? 0xffffffffu : (mul == 2 ? 0x00ff00ffu : 0x000000ffu);
    P.sel_odd = mul <= 4 ? P.sel : 0u;
    P.sel_rest = mul <= 8 ? P.sel : 0u;
    return P;
}

template <int NL>
static hipError_t launch_lists_n(const ListArgs<NL> &a, const uint8_t *mask_in, int32_t *block_counts, hipStream_t s)
{
    bool longer = false;
    int64_t most = 0;
    for (int l = 0; l < a.lists; ++l) {
        const LabelMap &L = a.at[l];
        longer = longer || (L.identity && (a.vec_in || L.packed_in) && compact_blocks(L.m) > kLongBlocks);
        most = L.m > most ? L.m : most;
    }
    bool once = most <= 16 * (int64_t)kOncePieces, brief = true; // (a read holds sixteen positions at most)
    RowPiecesArgs<NL> by_row;
    for (int l = 0; once && l < a.lists; ++l) {
        const LabelMap &L = a.at[l];
        const RowPieces &P = by_row.at[l] = row_pieces(L);
        const bool fast = L.identity && a.vec_in && !L.packed_in;
        const int64_t rows = ((int64_t)L.m + L.wl - 1) / L.wl;
        const int64_t reads = fast ? ((int64_t)L.m + 15) / 16 : rows * P.pieces * (L.w0 % 16 || L.col.add % 16 ? 2 : 1);
        if (fast || P.pieces > 0) {
            once = reads <= (fast ? kOncePieces : kOncePiecesStepped);
            brief = brief && reads <= kBriefPieces;
        } else {
            once = compact_blocks(L.m) <= kOnceBlocks;
            brief = brief && L.m <= 1024;
        }
    }
    if (once && brief) {
        hipLaunchKernelGGL((k_lists_once<NL, 256>), dim3((unsigned)((most + 1023) / 1024), a.lists), dim3(256), 0, s, a, by_row, mask_in);
        return hipGetLastError();
    }
    if (once) {
        hipLaunchKernelGGL((k_lists_once<NL, kListThreads>), dim3((unsigned)compact_blocks(most), a.lists), dim3(kListThreads), 0, s, a, by_row, mask_in);
        return hipGetLastError();
    }
    const int threads = longer ? kThreadsOf<16> : kThreadsOf<4>;
    hipLaunchKernelGGL((longer ? k_lists_count<NL, 16> : k_lists_count<NL, 4>), dim3(a.blocks), dim3(threads), 0, s, a,
                       mask_in, block_counts);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((longer ? k_lists_scatter<NL, 16> : k_lists_scatter<NL, 4>), dim3(a.blocks), dim3(threads), 0, s, a,
                       mask_in, (const int32_t *)block_counts);
    return hipGetLastError();
}

hipError_t launch_lists(const ListArgs<1> &a, const uint8_t *mask_in, int32_t *block_counts, hipStream_t s)
{
    return launch_lists_n(a, mask_in, block_counts, s);
}

hipError_t launch_lists(const ListArgs<kMaxPyramidLevels> &a, const uint8_t *mask_in, int32_t *block_counts, hipStream_t s)
{
    // (few pyramids have more: fewer arguments to hand over)
    constexpr int kFew = 5;
    if (a.lists > kFew) return launch_lists_n(a, mask_in, block_counts, s);
    ListArgs<kFew> few;
    few.lists = a.lists;
    few.blocks = a.blocks;
    few.vec_in = a.vec_in;
    few.ex = a.ex;
    for (int l = 0; l < a.lists; ++l) few.at[l] = a.at[l];
    return launch_lists_n(few, mask_in, block_counts, s);
}

static int32_t to_int32(int64_t v)
{
    const int64_t most = 1 << 30; // (far outside every image: what matters is the side it is clamped to)
    return (int32_t)(v > most ? most : (v < -most ? -most : v));
}

AxisMap compose_axis(int32_t stride, int32_t first, int32_t inner_size, const AxisMap &inner)
{
    auto image = [&](int64_t v) {
        const int64_t t = v * inner.mul + inner.add;
        return (int32_t)(t < inner.lo ? inner.lo : (t > inner.hi ? inner.hi : t));
    };
    AxisMap r;
    r.mul = to_int32((int64_t)stride * inner.mul);
    r.add = to_int32((int64_t)first * inner.mul + inner.add);
    r.lo = image(0);
    r.hi = image(inner_size - 1);
    return r;
}

hipError_t launch_compact(const MaskGeom &g, const uint8_t *mask_in, uint8_t *mask_out, int32_t *idx,
                          int32_t *count, int32_t *block_counts, const CompactExtras &extras, hipStream_t s)
{
    ListArgs<1> a;
    a.lists = 1;
    a.blocks = (int)compact_blocks(g.m);
    a.vec_in = (reinterpret_cast<uintptr_t>(mask_in) & 15u) == 0;
    a.ex = extras;
    LabelMap &L = a.at[0];
    L.m = (int32_t)g.m;
    L.hl = g.ho; L.wl = g.wo; L.h0 = g.h; L.w0 = g.w;
    L.identity = g.identity;
    L.packed_in = g.packed_in; L.packed_out = g.packed_out;
    L.block0 = 0;
    const AxisMap rows = {1, 0, 0, g.h - 1}, cols = {1, 0, 0, g.w - 1};
    L.row = compose_axis(g.sh, g.ch0, g.h, rows);
    L.col = compose_axis(g.sw, g.cw0, g.w, cols);
    L.div_w = make_fastdiv((uint32_t)g.wo);
    L.div_h = make_fastdiv((uint32_t)g.ho);
    L.mask_out = mask_out; L.idx = idx; L.count = count;
    return launch_lists(a, mask_in, block_counts, s);
}

// ---------------------------------------------------------------------------
// Kept positions in tile order (Sec. III-A fixes which patches become columns, not their
// order): tiles of tile_h x tile_w positions, row-major over the tiles of an image, row-major
// inside a tile.  A thread owns one row of one tile (up to 32 positions), a block 256 such rows
// in list order; two launches: per-block counts, then offsets + ordered scatter.
// ---------------------------------------------------------------------------
struct TiledGeom {
    int32_t n, ho, wo, th, tw, tiles_y, tiles_x;
    int32_t rows; // n * tiles_y * tiles_x * th tile rows (those below the image are empty)
};

// bit j = position (row of a tile, column j) is kept; *first = flat position of column 0
__device__ __forceinline__ uint32_t tiled_row_flags(const TiledGeom &g, const uint8_t *__restrict__ mask, int r,
                                                    int *first)
{
    *first = 0;
    if (r >= g.rows) return 0;
    const uint32_t t = (uint32_t)r / (uint32_t)g.th;
    const int dy = (int)((uint32_t)r - t * (uint32_t)g.th);
    const uint32_t t2 = t / (uint32_t)g.tiles_x;
    const int tx = (int)(t - t2 * (uint32_t)g.tiles_x);
    const int b = (int)(t2 / (uint32_t)g.tiles_y);
    const int ty = (int)(t2 - (uint32_t)b * (uint32_t)g.tiles_y);
    const int y = ty * g.th + dy, x0 = tx * g.tw;
    if (y >= g.ho) return 0;
    const int p = (b * g.ho + y) * g.wo + x0;
    *first = p;
    const int nx = min(g.tw, g.wo - x0);
    uint32_t flags = 0;
    if (nx == 16 && ((reinterpret_cast<uintptr_t>(mask) + (uintptr_t)p) & 15u) == 0) {
        const uint4 v = *reinterpret_cast<const uint4 *>(mask + p);
        const uint32_t wds[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int bb = 0; bb < 4; ++bb) flags |= ((wds[q] >> (8 * bb)) & 0xffu) ? (1u << (4 * q + bb)) : 0u;
    } else {
        uint8_t got[32];
#pragma unroll
        for (int j = 0; j < 32; ++j) got[j] = j < nx ? mask[p + j] : (uint8_t)0;
#pragma unroll
        for (int j = 0; j < 32; ++j) flags |= got[j] ? (1u << j) : 0u;
    }
    return flags;
}

__global__ __launch_bounds__(kCompactBlockThreads) void k_tiled_count(TiledGeom g, const uint8_t *__restrict__ mask,
                                                                       int32_t *__restrict__ block_counts)
{
    __shared__ int scratch[kCompactBlockThreads / 64];
    int first;
    const uint32_t flags = tiled_row_flags(g, mask, (int)(blockIdx.x * kCompactBlockThreads + threadIdx.x), &first);
    const int total = block_sum<kCompactBlockThreads / 64>(__popc(flags), scratch);
    if (threadIdx.x == 0) block_counts[blockIdx.x] = total;
}

__global__ __launch_bounds__(kCompactBlockThreads) void k_tiled_scatter(TiledGeom g, const uint8_t *__restrict__ mask,
                                                                         const int32_t *__restrict__ block_counts,
                                                                         int32_t *__restrict__ idx,
                                                                         int32_t *__restrict__ count)
{
    __shared__ int wave_sum[kCompactBlockThreads / 64];
    __shared__ int scratch[kCompactBlockThreads / 64];
    __shared__ int32_t stage[kCompactBlockThreads * 32];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int part = 0;
    for (int i = tid; i < (int)blockIdx.x; i += kCompactBlockThreads) part += block_counts[i];
    const int block_base = block_sum<kCompactBlockThreads / 64>(part, scratch);
    int first;
    const uint32_t flags = tiled_row_flags(g, mask, (int)(blockIdx.x * kCompactBlockThreads + tid), &first);
    const int c = __popc(flags);
    const int incl = wave_inclusive_scan(c);
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    int before = 0, block_total = 0;
#pragma unroll
    for (int i = 0; i < kCompactBlockThreads / 64; ++i) {
        if (i < wave) before += wave_sum[i];
        block_total += wave_sum[i];
    }
    int pos = before + incl - c;
    uint32_t f = flags;
    while (f) {
        const int j = __ffs(f) - 1;
        f &= f - 1;
        stage[pos++] = first + j;
    }
    __syncthreads();
    for (int i = tid; i < block_total; i += kCompactBlockThreads) idx[(int64_t)block_base + i] = stage[i];
    if (blockIdx.x == gridDim.x - 1 && tid == 0) *count = block_base + block_total;
}

hipError_t launch_compact_tiled(const uint8_t *mask, int n, int ho, int wo, int tile_h, int tile_w, int32_t *idx,
                                int32_t *count, int32_t *block_counts, hipStream_t s)
{
    TiledGeom g;
    g.n = n; g.ho = ho; g.wo = wo; g.th = tile_h; g.tw = tile_w;
    g.tiles_y = (ho + tile_h - 1) / tile_h;
    g.tiles_x = (wo + tile_w - 1) / tile_w;
    g.rows = n * g.tiles_y * g.tiles_x * tile_h;
    const int nb = (g.rows + kCompactBlockThreads - 1) / kCompactBlockThreads;
    hipLaunchKernelGGL(k_tiled_count, dim3(nb), dim3(kCompactBlockThreads), 0, s, g, mask, block_counts);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_tiled_scatter, dim3(nb), dim3(kCompactBlockThreads), 0, s, g, mask,
                       (const int32_t *)block_counts, idx, count);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Packed masks: one bit per pixel.  Packing: a thread turns sixteen bytes into sixteen bits.
// Rescaling (centre tap) between the two forms: sixteen output labels per thread.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_mask_rescale(MaskGeom g, const uint8_t *__restrict__ mask_in,
                                                      uint8_t *__restrict__ mask_out)
{
    const int64_t padded = g.packed_out ? ((g.m + 63) & ~(int64_t)63) : g.m;
    for (int64_t p0 = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 16; p0 < padded; p0 += (int64_t)gridDim.x * 256 * 16) {
        const uint32_t flags = kept_flags16(g, mask_in, p0);
        if (g.packed_out) {
            reinterpret_cast<uint16_t *>(mask_out)[p0 >> 4] = (uint16_t)flags;
        } else {
            for (int j = 0; j < 16 && p0 + j < g.m; ++j) mask_out[p0 + j] = (flags >> j) & 1u;
        }
    }
}

hipError_t launch_mask_rescale(const MaskGeom &g_in, const uint8_t *mask_in, uint8_t *mask_out, hipStream_t s)
{
    MaskGeom g = g_in;
    if (!g.packed_in && (reinterpret_cast<uintptr_t>(mask_in) & 15u)) g.identity = 0; // the 128-bit path needs alignment
    const int64_t threads = (g.m + 15) / 16 + 4;
    int64_t blocks = (threads + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_mask_rescale, dim3((unsigned)blocks), dim3(256), 0, s, g, mask_in, mask_out);
    return hipGetLastError();
}

hipError_t launch_mask_pack(const uint8_t *mask, int64_t m, uint64_t *bits, hipStream_t s)
{
    // a flat mask is a 1 x 1 x m image seen through a 1x1 stride-1 window
    MaskGeom g = mask_geom(1, 1, 1, 1, 1, 1, 1, 0, 0, 1, 1, 1, 1);
    g.w = g.wo = (int32_t)m;
    g.m = m;
    g.packed_out = 1;
    return launch_mask_rescale(g, mask, reinterpret_cast<uint8_t *>(bits), s);
}

// ---------------------------------------------------------------------------
// Zero-fill of the irrelevant output rows: a lane owns 16 bytes of one row.
// ---------------------------------------------------------------------------
// rows of whole 16-byte pieces
__global__ __launch_bounds__(256) void k_zero_fill16(Geom g, const uint8_t *__restrict__ mask_in,
                                                     const uint8_t *__restrict__ mask_out,
                                                     uint4 *__restrict__ out, int chunks_per_row)
{
    __shared__ int32_t dropped_s[4][64];
    const int wave = threadIdx.x >> 6;
    clear_irrelevant(g, mask_in, mask_out, out, chunks_per_row, (int)blockIdx.x * 4 + wave, (int)gridDim.x * 4,
                     dropped_s[wave]);
}

__global__ __launch_bounds__(256) void k_zero_fill_bytes(Geom g, const uint8_t *__restrict__ mask_in,
                                                         const uint8_t *__restrict__ mask_out,
                                                         uint8_t *__restrict__ out, int row_bytes)
{
    const int64_t total = (int64_t)g.m * row_bytes;
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < total;
         c += (int64_t)gridDim.x * blockDim.x) {
        const int64_t p = c / row_bytes;
        if (!position_kept(g, mask_in, mask_out, p)) out[c] = 0;
    }
}

hipError_t launch_zero_fill(const Geom &g, const uint8_t *mask_in, const uint8_t *mask_out, void *out,
                            int out_dtype, hipStream_t s)
{
    const int esz = out_dtype == FC_F32 ? 4 : (out_dtype == FC_FP8 ? 1 : 2);
    const int row_bytes = g.c_out * esz;
    if (row_bytes % 16 == 0) {
        const int cpr = row_bytes / 16;
        const int64_t groups = ((int64_t)g.m + 255) / 256; // 64 positions per wave, 4 waves per workgroup
        const int blocks = (int)(groups > 4096 ? 4096 : groups);
        hipLaunchKernelGGL(k_zero_fill16, dim3(blocks), dim3(256), 0, s, g, mask_in, mask_out, (uint4 *)out, cpr);
    } else {
        int64_t total = (int64_t)g.m * row_bytes;
        int blocks = (int)((total + 255) / 256 > 16384 ? 16384 : (total + 255) / 256);
        hipLaunchKernelGGL(k_zero_fill_bytes, dim3(blocks), dim3(256), 0, s, g, mask_in, mask_out, (uint8_t *)out,
                           row_bytes);
    }
    return hipGetLastError();
}

// Small fill kernel (a kernel rather than a memset node, so that callers can record it
// into HIP graphs).
__global__ __launch_bounds__(256) void k_zero_i32(int32_t *__restrict__ p, int n)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0;
}

hipError_t launch_zero_i32(int32_t *p, int n, hipStream_t s)
{
    hipLaunchKernelGGL(k_zero_i32, dim3((n + 255) / 256), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Max-pool helper (NHWC, whole tensor).  Padding never wins.
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void k_maxpool(const T *__restrict__ x, int n, int h, int w, int c, int k,
                                                 int stride, int pad, int ho, int wo,
                                                 const uint8_t *__restrict__ keep, T *__restrict__ out)
{
    const int64_t total = (int64_t)n * ho * wo * c;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        int ch = (int)(i % c);
        int64_t t = i / c;
        int ow = (int)(t % wo);
        t /= wo;
        int oh = (int)(t % ho);
        int b = (int)(t / ho);
        if (keep && !keep[((int64_t)b * ho + oh) * wo + ow]) {
            // a position the mask drops: no feature is computed for it (Sec. III-A); its window is not read
            T zero;
            __builtin_memset(&zero, 0, sizeof(T));
            out[i] = zero;
            continue;
        }
        bool have = false;
        float best = 0.f;
        T best_raw = x[0];
        for (int a = 0; a < k; ++a) {
            int ih = oh * stride - pad + a;
            if (ih < 0 || ih >= h) continue;
            for (int q = 0; q < k; ++q) {
                int iw = ow * stride - pad + q;
                if (iw < 0 || iw >= w) continue;
                T raw = x[(((int64_t)b * h + ih) * w + iw) * c + ch];
                float v = to_float(raw);
                if (!have || v > best) {
                    best = v;
                    best_raw = raw;
                    have = true;
                }
            }
        }
        out[i] = best_raw;
    }
}

// 16-bit types, channel count a multiple of 8: one lane owns 8 consecutive channels of an
// output position (16-byte loads and one 16-byte store).  IDX: the type the flat index is split
// in (32 bits whenever the tensor allows: the three divisions are most of the arithmetic).  K: window
// size known here (2, 3; all loads of a window in flight together: a small pool is a chain of round trips
// otherwise, 64 channels of one 112 x 112 map 7.2 us), or 0 = k.
template <typename T, typename IDX, int K>
__global__ __launch_bounds__(256) void k_maxpool_x8(const T *__restrict__ x, int n, int h, int w, int c, int k,
                                                    int stride, int pad, int ho, int wo,
                                                    const uint8_t *__restrict__ keep, T *__restrict__ out)
{
    const int cg = c / 8;
    const int64_t total = (int64_t)n * ho * wo * cg;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        IDX t = (IDX)i / (IDX)cg;
        const int g8 = (int)((IDX)i - t * (IDX)cg);
        const IDX pos = t; // (b * ho + oh) * wo + ow
        const IDX t2 = t / (IDX)wo;
        const int ow = (int)(t - t2 * (IDX)wo);
        const int b = (int)(t2 / (IDX)ho);
        const int oh = (int)(t2 - (IDX)b * (IDX)ho);
        if (keep && !keep[pos]) {
            *reinterpret_cast<uint4 *>(out + i * 8) = make_uint4(0, 0, 0, 0);
            continue;
        }
        bool have = false;
        float best[8];
        uint16_t raw[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            best[e] = 0.f;
            raw[e] = 0;
        }
        auto take = [&](const uint4 &v) __attribute__((always_inline)) {
            const uint32_t wd[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                T one;
                one.bits = (uint16_t)(wd[e >> 1] >> (16 * (e & 1)));
                const float f = to_float(one);
                if (!have || f > best[e]) {
                    best[e] = f;
                    raw[e] = one.bits;
                }
            }
            have = true;
        };
        const T *xb = x + (int64_t)b * h * w * c + g8 * 8;
        if constexpr (K > 0) {
            uint4 v[K * K];
            bool in[K * K];
#pragma unroll
            for (int a = 0; a < K; ++a)
#pragma unroll
                for (int q = 0; q < K; ++q) {
                    const int ih = oh * stride - pad + a, iw = ow * stride - pad + q;
                    in[a * K + q] = ih >= 0 && ih < h && iw >= 0 && iw < w;
                    // (a tap outside reads the nearest pixel inside and is dropped)
                    v[a * K + q] = *reinterpret_cast<const uint4 *>(
                        xb + (int64_t)(min(max(ih, 0), h - 1) * w + min(max(iw, 0), w - 1)) * c);
                }
#pragma unroll
            for (int t = 0; t < K * K; ++t)
                if (in[t]) take(v[t]);
        } else {
            for (int a = 0; a < k; ++a) {
                const int ih = oh * stride - pad + a;
                if (ih < 0 || ih >= h) continue;
                for (int q = 0; q < k; ++q) {
                    const int iw = ow * stride - pad + q;
                    if (iw < 0 || iw >= w) continue;
                    take(*reinterpret_cast<const uint4 *>(xb + (int64_t)(ih * w + iw) * c));
                }
            }
        }
        uint4 o;
        o.x = raw[0] | ((uint32_t)raw[1] << 16);
        o.y = raw[2] | ((uint32_t)raw[3] << 16);
        o.z = raw[4] | ((uint32_t)raw[5] << 16);
        o.w = raw[6] | ((uint32_t)raw[7] << 16);
        *reinterpret_cast<uint4 *>(out + i * 8) = o;
    }
}

// Grouped weights [c_out][taps][c_in / groups] written as the block-diagonal weights
// [c_out][taps][c_in] of the full layer that computes the same thing (zeros outside the
// blocks); esize = bytes per value.  One thread per output value.
__global__ __launch_bounds__(256) void k_expand_group_weights(const uint8_t *__restrict__ wg, int c_in, int c_out,
                                                              int taps, int groups, int esize,
                                                              uint8_t *__restrict__ wd)
{
    const int cig = c_in / groups, cog = c_out / groups;
    const int64_t total = (int64_t)c_out * taps * c_in;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int ci = (int)(i % c_in);
        const int64_t ct = i / c_in; // co * taps + tap
        const int co = (int)(ct / taps);
        const int grp = co / cog;
        const int cl = ci - grp * cig;
        const bool inside = cl >= 0 && cl < cig;
        for (int b = 0; b < esize; ++b) wd[i * esize + b] = inside ? wg[(ct * cig + cl) * esize + b] : (uint8_t)0;
    }
}

hipError_t launch_expand_group_weights(const void *wg, int c_in, int c_out, int taps, int groups, int esize,
                                       void *wd, hipStream_t s)
{
    const int64_t total = (int64_t)c_out * taps * c_in;
    const int blocks = (int)((total + 255) / 256 > 65536 ? 65536 : (total + 255) / 256);
    hipLaunchKernelGGL(k_expand_group_weights, dim3(blocks), dim3(256), 0, s, (const uint8_t *)wg, c_in, c_out, taps,
                       groups, esize, (uint8_t *)wd);
    return hipGetLastError();
}

hipError_t launch_maxpool(const void *x, int n, int h, int w, int c, int dtype, int k, int stride, int pad,
                          int ho, int wo, const uint8_t *keep, void *out, hipStream_t s)
{
    if (dtype != FC_F32 && c % 8 == 0) {
        const int64_t total8 = (int64_t)n * ho * wo * (c / 8);
        const int blocks8 = (int)((total8 + 255) / 256 > 65536 ? 65536 : (total8 + 255) / 256);
        const bool small = total8 < (int64_t)INT32_MAX;
#define FC_POOL(T, IDX, K)                                                                                         \
    hipLaunchKernelGGL((k_maxpool_x8<T, IDX, K>), dim3(blocks8), dim3(256), 0, s, (const T *)x, n, h, w, c, k, stride, \
                       pad, ho, wo, keep, (T *)out)
#define FC_POOL_T(T)                                       \
    if (!small) FC_POOL(T, int64_t, 0);                    \
    else if (k == 2) FC_POOL(T, uint32_t, 2);              \
    else if (k == 3) FC_POOL(T, uint32_t, 3);              \
    else FC_POOL(T, uint32_t, 0)
        if (dtype == FC_BF16) {
            FC_POOL_T(bf16_t);
        } else {
            FC_POOL_T(f16_t);
        }
#undef FC_POOL_T
#undef FC_POOL
        return hipGetLastError();
    }
    const int64_t total = (int64_t)n * ho * wo * c;
    int blocks = (int)((total + 255) / 256 > 65536 ? 65536 : (total + 255) / 256);
    if (dtype == FC_F32)
        hipLaunchKernelGGL(k_maxpool<float>, dim3(blocks), dim3(256), 0, s, (const float *)x, n, h, w, c, k, stride,
                           pad, ho, wo, keep, (float *)out);
    else if (dtype == FC_BF16)
        hipLaunchKernelGGL(k_maxpool<bf16_t>, dim3(blocks), dim3(256), 0, s, (const bf16_t *)x, n, h, w, c, k,
                           stride, pad, ho, wo, keep, (bf16_t *)out);
    else
        hipLaunchKernelGGL(k_maxpool<f16_t>, dim3(blocks), dim3(256), 0, s, (const f16_t *)x, n, h, w, c, k, stride,
                           pad, ho, wo, keep, (f16_t *)out);
    return hipGetLastError();
}

} // namespace fc
