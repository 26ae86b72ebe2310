// Focused convolution on the matrix cores for layers with very few input channels
// (RGB stems: C_in <= 4, K = KH*KW*C_in small).  Sec. III-A: only the kept patches
// become columns of the product.
//
// Such a layer is far too thin for the gather of the wide-layer kernel (a pixel is 6 bytes,
// not a 128-byte chunk), but its whole reduction fits a handful of 16-wide MFMA steps.  So
// the patch of a kept position is gathered element by element straight into the MFMA's
// B-operand registers: lane l of a wave owns position l % 32 of its 32-row block and the
// reduction elements (l / 32) * 8 .. + 8 of every 16-wide step; a small table in LDS gives,
// for each reduction index, the tap number and the element offset from the position's first tap.
// The pixels of one kernel row lie side by side, so the reduction is laid out kernel row by kernel
// row, each padded to whole pieces of 8 elements, and a lane fetches a piece with one (unaligned)
// 16-byte load; elements of taps outside the image or on an irrelevant input pixel, and
// the padding, are then replaced by zeros.  (7x7 on one 224 x 224 image: eight 2-byte loads a step
// and a weight loop with one load in flight took 32 us.)  Pieces that would reach past either end of x are loaded inside it and shifted: the
// first and the last image rows have such waves, and while these loaded element by element the launch lasted as long as they did (one
// 224 x 224 image 10.6 -> 9.1 us, 160 x 160 without a mask 12.5 -> 8.6).  A dilated kernel, and kernels whose rows are far from whole pieces load element by element -
// but for those of up to 4 x 4 taps with rows of at least 7 elements (3x3 RGB): their pieces, in plain order, lie in one
// kernel row or two and are put together from two 16-byte loads (TWO: two loads instead of eight, masks by four
// bytes, 10 registers fewer; 64 channels at 8 x 1080 x 1920, half kept: 507 -> 438 us, 32 at 32 x 224 x 224 / 2 without
// the zero-fill 14.9 -> 12.9 us).  The weights of 64 output channels sit in LDS as the A operand for the whole kernel; accumulators start from the bias; the epilogue
// applies ReLU, rounds once, transposes the tile through LDS and stores whole 16-byte row pieces.
// With a mask the kernel also clears the irrelevant rows: workgroups without a tile do it when
// there are enough of them, else all after their tiles.
#include "fc_mfma_util.hpp"
#include <algorithm>

namespace fc {

constexpr int kStemThreads = 256;   // 4 waves, 32 positions each
constexpr int kStemRows = 128;      // positions per tile
constexpr int kStemCo = 64;         // output channels per workgroup
constexpr int kStemMaxK = 160;      // longest reduction (7x7x3 = 147)
constexpr int kStemMaxPadded = 192; // longest reduction laid out by kernel rows (7 x 24 = 168)
constexpr int kStemMaxTaps = 64;    // tap-valid bits live in one 64-bit word per position

// bytes per weight row in LDS: the padded reduction plus one 16-byte piece, so that the 32
// rows a wave reads together start in different banks
__host__ __device__ static inline int stem_weight_pitch(int ksteps) { return ksteps * 32 + 16; }

bool conv_stem_supported(const Geom &g, int in_dtype, int out_dtype)
{
    if (in_dtype != FC_BF16 && in_dtype != FC_F16) return false;
    if (out_dtype != in_dtype && out_dtype != FC_F32 && out_dtype != FC_FP8) return false;
    if (g.c_in > 4 || g.c_out % 8 != 0) return false;
    if (out_dtype == FC_FP8 && g.c_out % 16 != 0) return false; // rows are stored in 16-byte pieces
    if (g.kh * g.kw > kStemMaxTaps || (g.kh * g.kw * g.c_in + 15) / 16 * 16 > kStemMaxK) return false;
    // element offset of the last tap from the first one, packed into 24 bits of a table entry
    const int64_t far = ((int64_t)(g.kh - 1) * g.dh * g.w + (int64_t)(g.kw - 1) * g.dw) * g.c_in + g.c_in;
    if (far >= (1 << 24)) return false;
    if ((int64_t)(g.kh - 1) * g.dh >= 65536 || (int64_t)(g.kw - 1) * g.dw >= 65536) return false; // 16-bit tap offsets
    if ((int64_t)g.n * g.h * g.w * g.c_in >= INT32_MAX) return false; // 32-bit element indices
    return true;
}

// Eight elements from element `off` on, where some lie before or past the tensor: loaded inside it and moved to their places (what takes
// the places of the others is never used).
__device__ __forceinline__ uint4 load8_moved(const uint16_t *__restrict__ x, int off, int elems)
{
    const int at = min(max(off, 0), elems - 8), up = at - off;
    uint64_t v[2];
    __builtin_memcpy(v, x + at, 16);
    const uint32_t n = (uint32_t)(up < 0 ? -up : up) * 16u;
    if (n != 0 && n < 128u) {
        const uint32_t r = n & 63u;
        if (up > 0) {
            v[1] = n < 64u ? (v[1] << r) | (v[0] >> (64u - r)) : v[0] << r;
            v[0] = n < 64u ? v[0] << r : 0u;
        } else {
            v[0] = n < 64u ? (v[0] >> r) | (v[1] << (64u - r)) : v[1] >> r;
            v[1] = n < 64u ? v[1] >> r : 0u;
        }
    }
    uint4 out;
    __builtin_memcpy(&out, v, 16);
    return out;
}

// divisors and the layout of the reduction, prepared on the host
struct StemDivs {
    FastDiv wo, ho, row;
    FastDiv per_co, per_row; // pieces of 8 elements: of the whole padded reduction, of one padded row
    int32_t row_pieces;
    int32_t pitch;  // padded elements of a kernel row; 0: reduction elements in plain (kh, kw, ci) order
    int32_t ksteps; // 16-wide steps of the (padded) reduction
    int32_t reach;  // elements from a position's first one to the end of its last piece
};

// Waves per SIMD: four fit the two-load form (118 registers); held to four, the other one spills (128 registers, 12 bytes a
// lane), with three it has the 143 it wants: 7x7 on 32 x 224 x 224 / 2, half kept, a list given: 35.5 -> 34.3 us, one image
// unchanged.
template <int DT, typename TO, bool TWO>
__global__ __launch_bounds__(kStemThreads, TWO ? 4 : 3) void k_conv_stem(
    Geom g, StemDivs dv, const uint16_t *__restrict__ x, const uint8_t *__restrict__ mask_in,
    const uint8_t *__restrict__ mask_out, const uint16_t *__restrict__ w, const float *__restrict__ bias,
    const int32_t *__restrict__ idx, const int32_t *__restrict__ count, TO *__restrict__ out)
{
    constexpr int OP = kStemCo * (int)sizeof(TO) + 16;         // bytes per output row in LDS
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5;
    const int rows = idx ? *count : g.m;
    const int taps = g.kh * g.kw;
    const int K = taps * g.c_in;
    const int ksteps = dv.ksteps;
    const int row_len = g.kw * g.c_in; // reduction elements of a kernel row
    // LDS, sized by the launcher for this layer's reduction length (a 3x3x3 stem needs 24 KB,
    // so six workgroups share a CU and hide each other's gather latency)
    const int WPITCH = stem_weight_pitch(ksteps);                   // bytes per weight row
    extern __shared__ __align__(16) unsigned char stem_lds[];
    unsigned char *o_s = stem_lds;                                  // [rows][OP]
    unsigned char *w_s = o_s + kStemRows * OP;                      // [channel][k] as stored
    uint32_t *lut = reinterpret_cast<uint32_t *>(w_s + kStemCo * WPITCH); // tap << 24 | element offset
    int32_t *row_p = reinterpret_cast<int32_t *>(lut + ksteps * 16);
    float *bias_s = reinterpret_cast<float *>(row_p + kStemRows);   // [channel]
    uint32_t *tap_s = reinterpret_cast<uint32_t *>(bias_s + kStemCo); // [tap] kh*dh | kw*dw << 16
    uint4 *piece_s = reinterpret_cast<uint4 *>(tap_s + kStemMaxTaps); // two_rows: three words of four per piece, see below
    const int co0 = blockIdx.y * kStemCo;

    // ---- once per workgroup: weights, a piece of 8 reduction elements per load, and the
    // reduction-index table ----
    {
        const int per_co = ksteps * 2, w_elems = g.c_out * K;
        const int wrow = dv.pitch ? row_len : K; // elements of a padded row
        constexpr int U = 3; // loads in flight
        for (int i0 = tid; i0 < kStemCo * per_co; i0 += U * kStemThreads) {
            uint4 wv[U];
            int left[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = i0 + u * kStemThreads;
                const int j = (int)fast_div((uint32_t)i, dv.per_co), q = i - j * per_co;
                const int row = (int)fast_div((uint32_t)q, dv.per_row), e0 = (q - row * dv.row_pieces) * 8;
                // elements of the piece that exist; one that would leave the tensor is loaded further up
                left[u] = (j < kStemCo && co0 + j < g.c_out && row * wrow < K) ? min(wrow - e0, 8) : 0;
                const int src = left[u] > 0 ? (co0 + j) * K + row * wrow + e0 : 0, at = min(src, w_elems - 8);
                left[u] |= (src - at) << 8;
                __builtin_memcpy(&wv[u], w + at, 16);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = i0 + u * kStemThreads;
                const int n = left[u] & 255;
                for (int k = left[u] >> 8; k > 0; --k) { // ... and moved back, an element at a time (rare)
                    wv[u].x = (wv[u].x >> 16) | (wv[u].y << 16);
                    wv[u].y = (wv[u].y >> 16) | (wv[u].z << 16);
                    wv[u].z = (wv[u].z >> 16) | (wv[u].w << 16);
                    wv[u].w >>= 16;
                }
                auto keep = [&](int t) { return t + 1 < n ? 0xffffffffu : (t < n ? 0xffffu : 0u); };
                const uint4 v = make_uint4(wv[u].x & keep(0), wv[u].y & keep(2), wv[u].z & keep(4), wv[u].w & keep(6));
                const int j = (int)fast_div((uint32_t)i, dv.per_co), q = i - j * per_co;
                if (j < kStemCo) *reinterpret_cast<uint4 *>(w_s + j * WPITCH + q * 16) = v;
            }
        }
    }
    for (int k = tid; k < ksteps * 16; k += kStemThreads) {
        uint32_t e = 0xff000000u; // padding of the reduction: a tap number no position has (63 modulo 64)
        const int kh = dv.pitch ? k / dv.pitch : (int)fast_div((uint32_t)k, dv.row);
        const int r = k - kh * (dv.pitch ? dv.pitch : row_len);
        if (kh < g.kh) {
            const int kw = r / g.c_in, ci = r - kw * g.c_in;
            // (the first element of a piece carries its offset whether or not it is padding)
            e = (uint32_t)((kh * g.dh * g.w + kw * g.dw) * g.c_in + ci) |
                (r < row_len ? (uint32_t)(kh * g.kw + kw) << 24 : 0xff000000u);
        }
        lut[k] = e;
    }
    if (tid < kStemCo) bias_s[tid] = (bias && co0 + tid < g.c_out) ? bias[co0 + tid] : 0.f;
    if (tid < kStemMaxTaps) {
        const int kh = tid / g.kw, kw = tid - kh * g.kw;
        tap_s[tid] = tid < taps ? (uint32_t)(kh * g.dh) | ((uint32_t)(kw * g.dw) << 16) : 0u;
    }
    // A piece of 8 elements in plain order lies in one kernel row or in two: it is then put together from two loads,
    // the second one starting as many elements early as the first contributes.  Per piece: halves that come from
    // the first, tap pairs (low | high << 16; padding: tap 31, which no such layer has), the two element offsets.
    if (TWO && tid < ksteps * 2) {
        const int e0 = tid * 8, row = (int)fast_div((uint32_t)e0, dv.row), in_row = e0 - row * row_len;
        const int first = min(row_len - in_row, 8);
        uint32_t from_first[4], pair[4];
        for (int q = 0; q < 4; ++q) {
            from_first[q] = (2 * q < first ? 0xffffu : 0u) | (2 * q + 1 < first ? 0xffff0000u : 0u);
            pair[q] = 0;
            for (int h = 0; h < 2; ++h) {
                const int k = e0 + 2 * q + h;
                pair[q] |= (uint32_t)(k < K ? k / g.c_in : 31) << (16 * h);
            }
        }
        const int at = row * g.dh * g.w * g.c_in + in_row, next = (row + 1) * g.dh * g.w * g.c_in - first;
        const bool some = e0 < K, both = first < 8 && row + 1 < g.kh;
        piece_s[tid * 3] = make_uint4(from_first[0], from_first[1], from_first[2], from_first[3]);
        piece_s[tid * 3 + 1] = make_uint4(pair[0], pair[1], pair[2], pair[3]);
        piece_s[tid * 3 + 2] = make_uint4(some ? (uint32_t)at : 0u, some && both ? (uint32_t)next : (some ? (uint32_t)at : 0u), 0u, 0u);
    }
    __syncthreads();
    const uint64_t all_taps = taps >= 64 ? ~0ull : ((1ull << taps) - 1ull);
    const int reach_h = (g.kh - 1) * g.dh, reach_w = (g.kw - 1) * g.dw;

    const int ntiles = (rows + kStemRows - 1) / kStemRows;
    // ---- locating a tile's rows, in pieces so that the memory round trips of the NEXT tile
    // (position list, then mask bytes) run under the gathers, MFMAs and stores of the current
    // one.  Piece 1: the list entry.  Piece 2: decode it and request the mask bytes, the taps of a
    // kernel row with one (unaligned) 8-byte load, alternate kernel rows per half-wave.  Piece 3: tap-valid
    // bits from those bytes, halves merged.  (Kernels with more than eight rows or columns, or
    // dilated: tap by tap in piece 3.) ----
    const int64_t mask_bytes = (int64_t)g.n * g.h * g.w;
    const bool by_rows = g.kw <= 8 && g.kh <= 8 && g.dw == 1 && mask_bytes >= 8;
    struct Located {
        int p, base, ih0, iw0, b;
        bool lookup;       // bits have to be built
        uint2 rows[TWO ? 1 : 4];
        uint32_t row4[TWO ? 2 : 1]; // TWO: four bytes of kernel rows half and half + 2
    };
    auto fetch_entry = [&](int tile) -> int {
        const int r = tile * kStemRows + wave * 32 + (lane & 31);
        return r < rows ? (idx ? idx[r] : r) : -1;
    };
    auto decode = [&](int p, Located &L) {
        L.p = p;
        L.base = 0;
        L.ih0 = L.iw0 = L.b = 0;
        L.lookup = false;
        if (p >= 0) {
            const int q = (int)fast_div((uint32_t)p, dv.wo);
            const int ow = p - q * g.wo;
            L.b = (int)fast_div((uint32_t)q, dv.ho);
            const int oh = q - L.b * g.ho;
            L.ih0 = oh * g.sh - g.ph;
            L.iw0 = ow * g.sw - g.pw;
            L.base = ((L.b * g.h + L.ih0) * g.w + L.iw0) * g.c_in; // may point before the image: only used with a valid tap
            const bool interior = L.ih0 >= 0 && L.ih0 + reach_h < g.h && L.iw0 >= 0 && L.iw0 + reach_w < g.w;
            L.lookup = mask_in || !interior; // else every tap is inside the image and nothing gates it
        }
        if constexpr (TWO) {
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                L.row4[v] = 0x01010101u;
                if (mask_in && half + 2 * v < g.kh) {
                    const int off = (L.b * g.h + L.ih0 + (half + 2 * v) * g.dh) * g.w + L.iw0; // (positions fit 31 bits)
                    const int at = min(max(off, 0), (int)mask_bytes - 4), moved = off - at;
                    uint32_t m;
                    __builtin_memcpy(&m, mask_in + at, 4);
                    L.row4[v] = moved < 0 ? (moved > -4 ? m << (-8 * moved) : 0u) : (moved < 4 ? m >> (8 * moved) : 0u);
                }
            }
        } else if (by_rows) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                L.rows[v] = make_uint2(0x01010101u, 0x01010101u);
                if (mask_in && 2 * v < g.kh) {
                    // bytes from the row's first tap on; a load that would leave the mask is moved inside
                    // it and its bytes moved back (what lies outside the image is dropped below)
                    const int64_t off = (int64_t)(L.b * g.h + L.ih0 + (half + 2 * v) * g.dh) * g.w + L.iw0;
                    const int64_t at = off < 0 ? 0 : (off > mask_bytes - 8 ? mask_bytes - 8 : off);
                    uint64_t m;
                    __builtin_memcpy(&m, mask_in + at, 8);
                    const int64_t moved = off - at;
                    m = moved < 0 ? (moved > -8 ? m << (-8 * moved) : 0ull) : (moved < 8 ? m >> (8 * moved) : 0ull);
                    L.rows[v] = make_uint2((uint32_t)m, (uint32_t)(m >> 32));
                }
            }
        }
    };
    auto finish = [&](const Located &L) -> uint64_t {
        if (!L.lookup) return L.p >= 0 ? all_taps : 0ull;
        uint64_t bits = 0;
        if (TWO || by_rows) {
            // columns of the kernel inside the image
            const int c0 = max(-L.iw0, 0), c1 = min(g.w - L.iw0, g.kw); // [c0, c1)
            const uint32_t cols = c1 > c0 ? ((1u << c1) - 1u) & ~((1u << c0) - 1u) : 0u;
            auto four = [](uint32_t v) { // one bit per nonzero byte
                v = (((v & 0x7f7f7f7fu) + 0x7f7f7f7fu) | v) & 0x80808080u;
                return ((v >> 7) & 1u) | ((v >> 14) & 2u) | ((v >> 21) & 4u) | (v >> 28);
            };
            if constexpr (TWO) {
                uint32_t low = 0;
#pragma unroll
                for (int v = 0; v < 2; ++v) {
                    const int kh = half + 2 * v, ih = L.ih0 + kh * g.dh;
                    if (kh < g.kh && (uint32_t)ih < (uint32_t)g.h) low |= (four(L.row4[v]) & cols) << (kh * g.kw);
                }
                return low | (uint32_t)__shfl_xor((int)low, 32, 64);
            } else {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int kh = half + 2 * v, ih = L.ih0 + kh * g.dh;
                const bool in = kh < g.kh && (uint32_t)ih < (uint32_t)g.h;
                const uint32_t r = in ? (four(L.rows[v].x) | (four(L.rows[v].y) << 4)) & cols : 0u;
                bits |= (uint64_t)r << ((kh * g.kw) & 63);
            }
            }
        } else {
            for (int t = half; t < taps; t += 2) {
                const uint32_t e = tap_s[t];
                const int ih = L.ih0 + (int)(e & 0xffffu), iw = L.iw0 + (int)(e >> 16);
                bool in = ih >= 0 && ih < g.h && iw >= 0 && iw < g.w;
                if (in && mask_in) in = mask_in[(int64_t)(L.b * g.h + ih) * g.w + iw] != 0;
                bits |= (uint64_t)in << t;
            }
        }
        // merge the halves' bits
        const uint32_t lo = (uint32_t)bits, hi = (uint32_t)(bits >> 32);
        const uint32_t lo2 = lo | (uint32_t)__shfl_xor((int)lo, 32, 64);
        const uint32_t hi2 = hi | (uint32_t)__shfl_xor((int)hi, 32, 64);
        return (uint64_t)lo2 | ((uint64_t)hi2 << 32);
    };

    const int x_elems = g.n * g.h * g.w * g.c_in;
    Located nxt;
    uint64_t bits_n = 0;
    if ((int)blockIdx.x < ntiles) {
        decode(fetch_entry(blockIdx.x), nxt);
        bits_n = finish(nxt);
    }
    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int p = nxt.p, base = nxt.base;
        const uint64_t bits = bits_n;
        const bool more = tile + (int)gridDim.x < ntiles;
        const int entry_n = more ? fetch_entry(tile + gridDim.x) : -1; // piece 1 of the next tile
        if (half == 0) row_p[wave * 32 + (lane & 31)] = p;

        f32x16_t acc[2];
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                // channel = cb*32 + (i/4)*8 + half*4 + i%4 of accumulator i
                const float4 bq = *reinterpret_cast<const float4 *>(bias_s + cb * 32 + q * 8 + half * 4);
                acc[cb][q * 4 + 0] = bq.x;
                acc[cb][q * 4 + 1] = bq.y;
                acc[cb][q * 4 + 2] = bq.z;
                acc[cb][q * 4 + 3] = bq.w;
            }

        auto selected = [&](uint32_t ent) { return ((ent >> 24) < (uint32_t)kStemMaxTaps) && ((bits >> ((ent >> 24) & 63u)) & 1ull); };
        // all ones in the halves whose element is in use (padding: tap 63, which no such layer has)
        auto pair_mask = [&](uint32_t lo, uint32_t hi) -> uint32_t {
            const uint32_t t = ((uint32_t)(bits >> ((lo >> 24) & 63u)) & 1u) | (((uint32_t)(bits >> ((hi >> 24) & 63u)) & 1u) << 16);
            return (t << 16) - t;
        };
        auto multiply = [&](int j, const uint4 &xf) {
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                const uint4 wf = *reinterpret_cast<const uint4 *>(w_s + (cb * 32 + (lane & 31)) * WPITCH +
                                                                   (j * 16 + half * 8) * 2);
                acc[cb] = mfma32<DT>(wf, xf, acc[cb]);
            }
        };
        const bool inside = __all(base >= 0 && base <= x_elems - dv.reach);
        if (!TWO && dv.pitch && x_elems >= 8) {
            constexpr int U = 4; // pieces in flight
            for (int j0 = 0; j0 < ksteps; j0 += U) {
                uint4 v[U];
                if (inside) {
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const uint32_t e = lut[min(j0 + u, ksteps - 1) * 16 + half * 8];
                        __builtin_memcpy(&v[u], x + base + (int)(e & 0xffffffu), 16);
                    }
                } else {
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        v[u] = load8_moved(x, base + (int)(lut[min(j0 + u, ksteps - 1) * 16 + half * 8] & 0xffffffu), x_elems);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (j0 + u >= ksteps) break;
                    const uint32_t *le = &lut[(j0 + u) * 16 + half * 8];
                    const uint4 e0 = *reinterpret_cast<const uint4 *>(le), e1 = *reinterpret_cast<const uint4 *>(le + 4);
                    uint4 xf;
                    xf.x = v[u].x & pair_mask(e0.x, e0.y);
                    xf.y = v[u].y & pair_mask(e0.z, e0.w);
                    xf.z = v[u].z & pair_mask(e1.x, e1.y);
                    xf.w = v[u].w & pair_mask(e1.z, e1.w);
                    multiply(j0 + u, xf);
                }
            }
        } else if (TWO && inside) {
            constexpr int U = 2; // steps in flight
            for (int j0 = 0; j0 < ksteps; j0 += U) {
                uint4 a[U], b[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint4 at = piece_s[(min(j0 + u, ksteps - 1) * 2 + half) * 3 + 2];
                    __builtin_memcpy(&a[u], x + base + (int)at.x, 16);
                    __builtin_memcpy(&b[u], x + base + (int)at.y, 16);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (j0 + u >= ksteps) break;
                    const uint4 f = piece_s[((j0 + u) * 2 + half) * 3], t = piece_s[((j0 + u) * 2 + half) * 3 + 1];
                    auto gate = [&](uint32_t pair) -> uint32_t { // all ones in the halves whose tap is valid
                        const uint32_t lo = (uint32_t)__builtin_amdgcn_sbfe((int)bits, pair & 31u, 1);
                        const uint32_t hi = (uint32_t)__builtin_amdgcn_sbfe((int)bits, (pair >> 16) & 31u, 1);
                        return (lo & 0xffffu) | (hi & 0xffff0000u);
                    };
                    uint4 xf;
                    xf.x = ((a[u].x & f.x) | (b[u].x & ~f.x)) & gate(t.x);
                    xf.y = ((a[u].y & f.y) | (b[u].y & ~f.y)) & gate(t.y);
                    xf.z = ((a[u].z & f.z) | (b[u].z & ~f.z)) & gate(t.z);
                    xf.w = ((a[u].w & f.w) | (b[u].w & ~f.w)) & gate(t.w);
                    multiply(j0 + u, xf);
                }
            }
        } else {
            for (int j = 0; j < ksteps; ++j) {
                // this lane's 8 reduction elements of step j
                const uint4 e0 = *reinterpret_cast<const uint4 *>(&lut[j * 16 + half * 8]);
                const uint4 e1 = *reinterpret_cast<const uint4 *>(&lut[j * 16 + half * 8 + 4]);
                const uint32_t ent[8] = {e0.x, e0.y, e0.z, e0.w, e1.x, e1.y, e1.z, e1.w};
                uint32_t val[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) val[e] = selected(ent[e]) ? (uint32_t)x[base + (int)(ent[e] & 0xffffffu)] : 0u;
                uint4 xf;
                xf.x = val[0] | (val[1] << 16);
                xf.y = val[2] | (val[3] << 16);
                xf.z = val[4] | (val[5] << 16);
                xf.w = val[6] | (val[7] << 16);
                multiply(j, xf);
            }
        }

        if (more) decode(entry_n, nxt); // piece 2 of the next tile: its mask bytes travel during the epilogue

        // ---- epilogue: ReLU, one rounding, transposed through LDS, 16-byte row pieces ----
        __syncthreads(); // the previous tile's stores have read o_s; row_p is complete
        const int rl = wave * 32 + (lane & 31);
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int cl = cb * 32 + q * 8 + half * 4;
                float v0 = acc[cb][q * 4 + 0], v1 = acc[cb][q * 4 + 1];
                float v2 = acc[cb][q * 4 + 2], v3 = acc[cb][q * 4 + 3];
                if constexpr (sizeof(TO) == 4) {
                    if (g.flags & FC_RELU) {
                        v0 = relu_keep_nan(v0); v1 = relu_keep_nan(v1);
                        v2 = relu_keep_nan(v2); v3 = relu_keep_nan(v3);
                    }
                    store4<DT, TO>(reinterpret_cast<TO *>(o_s + rl * OP) + cl, v0, v1, v2, v3);
                } else if constexpr (sizeof(TO) == 1) {
                    uint32_t pk;
                    store4<DT, TO>(reinterpret_cast<TO *>(&pk), v0, v1, v2, v3);
                    if (g.flags & FC_RELU) pk = relu_packed8(pk);
                    *reinterpret_cast<uint32_t *>(o_s + rl * OP + cl) = pk;
                } else {
                    uint2 pk;
                    store4<DT, TO>(reinterpret_cast<TO *>(&pk), v0, v1, v2, v3);
                    if (g.flags & FC_RELU) {
                        pk.x = relu_packed16(pk.x);
                        pk.y = relu_packed16(pk.y);
                    }
                    *reinterpret_cast<uint2 *>(o_s + rl * OP + cl * 2) = pk;
                }
            }
        __syncthreads();
        constexpr int PPR = kStemCo * (int)sizeof(TO) / 16; // 16-byte pieces per row
        constexpr int EPT = 16 / (int)sizeof(TO);
        for (int i = tid; i < kStemRows * PPR; i += kStemThreads) {
            const int rr = i / PPR, pc = i - rr * PPR;
            const int pp = row_p[rr];
            const int co = co0 + pc * EPT;
            if (pp >= 0 && co < g.c_out)
                __builtin_nontemporal_store(*reinterpret_cast<const u32x4_t *>(o_s + rr * OP + pc * 16),
                                            reinterpret_cast<u32x4_t *>(out + (int64_t)pp * g.c_out + co));
        }
        if (more) bits_n = finish(nxt); // piece 3
        __syncthreads(); // everyone is done with row_p and o_s before the next tile rewrites them
    }

    if (mask_in && !(g.flags & FC_SKIP_ZERO_FILL)) {
        const int idle = (int)gridDim.x - ntiles;
        const bool idle_only = idle >= (int)gridDim.x / 16 && idle > 0;
        const int me = idle_only ? (int)blockIdx.x - ntiles : (int)blockIdx.x, of = idle_only ? idle : (int)gridDim.x;
        if (me >= 0)
            clear_irrelevant(g, mask_in, mask_out, out, g.c_out * (int)sizeof(TO) / 16,
                             (me * (int)gridDim.y + (int)blockIdx.y) * (kStemThreads / 64) + wave,
                             of * (int)gridDim.y * (kStemThreads / 64), reinterpret_cast<int32_t *>(stem_lds) + wave * 64);
    }
}

template <int DT, typename TO>
static hipError_t launch_stem_t(const Geom &g, const void *x, const uint8_t *mask_in, const uint8_t *mask_out, const void *w,
                                const float *bias, const int32_t *idx, const int32_t *count, void *out,
                                hipStream_t s)
{
    // (the grid is sized below)
    const int64_t tiles = ((int64_t)g.m + kStemRows - 1) / kStemRows;
    const int gy = (g.c_out + kStemCo - 1) / kStemCo;
    StemDivs dv;
    dv.wo = make_fastdiv((uint32_t)g.wo);
    dv.ho = make_fastdiv((uint32_t)g.ho);
    dv.row = make_fastdiv((uint32_t)(g.kw * g.c_in));
    dv.pitch = (g.kw * g.c_in + 7) / 8 * 8;
    // short kernel rows are mostly padding (3x3x3: three steps for two): those keep the plain order
    if (g.dw != 1 || g.kh * dv.pitch > kStemMaxPadded || g.kh * g.kw > 63 ||
        4 * g.kh * dv.pitch > 5 * g.kh * g.kw * g.c_in)
        dv.pitch = 0;
    const int ksteps = dv.ksteps = ((dv.pitch ? g.kh * dv.pitch : g.kh * g.kw * g.c_in) + 15) / 16;
    dv.row_pieces = dv.pitch ? dv.pitch / 8 : ksteps * 2;
    dv.per_row = make_fastdiv((uint32_t)dv.row_pieces);
    dv.per_co = make_fastdiv((uint32_t)(ksteps * 2));
    // plain order: pieces of 8 elements that span at most two kernel rows, of kernels of up to 4 x 4 taps (an early
    // start of the second row's load stays behind the position's first element when an image row has 8)
    const bool two_rows = !dv.pitch && g.dw == 1 && g.kw * g.c_in >= 7 && g.kh <= 4 && g.kw <= 4 &&
                          g.w * g.c_in >= 8 && (int64_t)g.n * g.h * g.w >= 8;
    dv.reach = (g.kh - 1) * g.dh * g.w * g.c_in + (dv.pitch ? dv.pitch : g.kw * g.c_in + 8);
    const size_t lds = (size_t)kStemRows * (kStemCo * sizeof(TO) + 16) + (size_t)kStemCo * stem_weight_pitch(ksteps) +
                       (size_t)ksteps * 16 * sizeof(uint32_t) + (size_t)kStemRows * sizeof(int32_t) + (size_t)kStemCo * sizeof(float) +
                       (size_t)kStemMaxTaps * sizeof(uint32_t) + (two_rows ? (size_t)ksteps * 2 * 3 * sizeof(uint4) : 0);
    // Sized for the dense row count (the kept count is only known on the device), capped at the workgroups that are resident together:
    // they stride over the tiles, the next one's rows looked up beside the current one, and lay out the weights once.  At 2048 a
    // workgroup had one tile and its own weights, or a second round of workgroups was started for the rest.  us, half kept, lists given, other buffers each time,
    // 2048 -> resident: 3x3, 3 -> 64 on 2 x 360 x 640 without a mask 19.0 -> 17.3, zero-filled 23.4 -> 18.5, chained 16.2 -> 14.0, on 8 x 1080 x 1920 without a mask 426 ->
    // 423, chained 265 -> 266; 3 -> 32 on 32 x 224 x 224 / 2 16.7 -> 14.9, 15.7 -> 13.8, 14.4 -> 11.8; 7x7 / 2, 3 -> 64, on 32 x 224 x 224 37.3 -> 32.1, 31.6 -> 28.4,
    // 31.1 -> 25.0, on 16 x 1080 x 1920 518 -> 512, 419 -> 405, 360 -> 349.  512 or 1536 for the 3x3 layers 11 .. 34 % and 7 .. 19 % slower, 512 for the 7x7 ones 3 .. 32 %.
    // Workgroups that are done clear rows beside others' tiles only where more are started than are resident: kernels of few taps into more memory than the
    // last cache level, where clearing is much of the launch.  Zero-filled, 2048 -> resident: 3x3, 3 -> 64 on 3 x 600 x 800 (184 MB) 45.3 -> 44.7, on 2 x 720 x 1280
    // (236 MB) 55.9 -> 56.4, on 4 x 720 x 1280 107 -> 108.5, on 4 x 1080 x 1920 229 -> 239, on 8 of them 444 -> 463; 3 -> 128 on 2 x 360 x 640 (118 MB) 37.5 -> 31.5, on 2 x 600
    // x 800 (246 MB) 57.3 -> 60.3; 3 -> 32 on 1 x 1080 x 1920 (133 MB) 48.0 -> 46.4, on 2 (265 MB) 88.4 -> 89.3; / 2 on 16 x 720 x 1280 107 -> 109; 5x5, 3 -> 64 on 1 x 1080 x
    // 1920 (265 MB) 90.6 -> 86.1, on 4 (1 062 MB) 324 -> 332; 7x7 there 402 -> 397.
    const int64_t out_bytes = (int64_t)g.m * g.c_out * (int64_t)sizeof(TO);
    const bool beside = mask_in && !(g.flags & FC_SKIP_ZERO_FILL) && g.kh * g.kw <= 25 && out_bytes >= (int64_t)std::max(g.kh * g.kw, 9) * 22000000;
    const int resident = beside ? 2048 : conv_grid_cus() * (two_rows ? 4 : 3) / gy;
    const int gx = (int)std::min<int64_t>(tiles, std::max(resident, 1));
    auto kern = two_rows ? k_conv_stem<DT, TO, true> : k_conv_stem<DT, TO, false>;
    hipLaunchKernelGGL(kern, dim3(gx, gy), dim3(kStemThreads), lds, s, g, dv, (const uint16_t *)x,
                       mask_in, mask_out, (const uint16_t *)w, bias, idx, count, (TO *)out);
    return hipGetLastError();
}

hipError_t launch_conv_stem(const Geom &g, int in_dtype, int out_dtype, const void *x, const uint8_t *mask_in,
                            const uint8_t *mask_out, const void *w, const float *bias, const int32_t *idx,
                            const int32_t *count, void *out, hipStream_t s)
{
    if (in_dtype == FC_BF16) {
        if (out_dtype == FC_F32) return launch_stem_t<FC_BF16, float>(g, x, mask_in, mask_out, w, bias, idx, count, out, s);
        if (out_dtype == FC_FP8) return launch_stem_t<FC_BF16, uint8_t>(g, x, mask_in, mask_out, w, bias, idx, count, out, s);
        return launch_stem_t<FC_BF16, uint16_t>(g, x, mask_in, mask_out, w, bias, idx, count, out, s);
    }
    if (out_dtype == FC_F32) return launch_stem_t<FC_F16, float>(g, x, mask_in, mask_out, w, bias, idx, count, out, s);
    if (out_dtype == FC_FP8) return launch_stem_t<FC_F16, uint8_t>(g, x, mask_in, mask_out, w, bias, idx, count, out, s);
    return launch_stem_t<FC_F16, uint16_t>(g, x, mask_in, mask_out, w, bias, idx, count, out, s);
}

} // namespace fc
