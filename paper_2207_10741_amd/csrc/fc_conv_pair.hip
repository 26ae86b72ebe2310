// Two focused 1x1 layers one after the other on the gfx950 matrix cores, the second the only reader of the first: the
// feature map between them stays in registers.
//
// A chained network is full of such pairs: a bottleneck's expansion and the next one's reduction (64 -> 256 -> 64), an
// inverted residual's projection and the next one's expansion (192 -> 32 -> 192).  As two launches the wide map goes
// through memory twice, or the launch and its chain of round trips (count, list, rows) is paid twice for a few
// microseconds of work.  Both layers see the same kept rows (1x1, unit stride), so a wave that owns 32 rows needs
// nothing but the weights: those of both layers stay in LDS for the whole launch, and each wave is a pipeline of its own
// over units of 32 rows as in k_conv_pw (rows gathered by loads into LDS ahead of their use, no barrier after the prologue).
//
// The first layer's accumulators become the second one's operand without leaving the wave.  A lane of a product holds four
// runs of four channels of its row, the runs of the two lane halves interleaved; rounded and packed, one exchange between the halves
// (v_permlane32_swap) per packed register gives every lane the channels that the next product takes from it.  Operands, the order of the
// steps and the place where the bias is added are those of the kernel that serves each layer by itself, so the sums are the same
// bit for bit.
//
// What bounds it: the matrix and vector work of a unit (a block of the middle is 8 products and 40 vector instructions; 64 -> 256 -> 64
// on 32 x 120 x 160, half kept, moves 82 MB in 35 us) on large layers, round trips and the fetch of the weights on small ones.
// us, two launches -> one, half kept, inside a network: 64 -> 256 -> 64 on 32 x 120 x 160 35 + 43 -> 35, E4M3 32 + 20 -> 31; 32 -> 16 -> 96 on
// 32 x 112 x 112 9.2 + 14.7 -> 17.3; 144 -> 24 -> 144 on 32 x 56 x 56 8.4 + 9.4 -> 12.0; 192 -> 32 -> 192 on 32 x 28 x 28 5.0 + 7.4 -> 7.7;
// 384 -> 64 -> 384 on 32 x 14 x 14 6.2 + 7.0 -> 9.9.  By themselves, half kept: 64 -> 256 -> 64 on 2 x 14 x 14 9.7 -> 6.3, on 8 x 40 x 40 12.6 -> 7.2;
// 384 -> 64 -> 384 on 2 x 10 x 10 9.3 -> 8.5, on 64 x 28 x 28 19.4 -> 18.7 (the least); 32 -> 16 -> 96 on 64 x 112 x 112 45.9 -> 35.7.  Nothing loses: 110 pairs of
// random sizes, with a mask and without, 0.49 .. 1.00 of the two launches.
//
// WIDE: the middle is wider than the output (at most NB * 32 channels): the output's accumulators stay, the middle is made
// two blocks of 32 channels at a time.  Else the middle is at most NB * 32 channels: it is made whole, the output two blocks at
// a time.
#include "fc_dma_util.hpp"
#include <algorithm>
#include <atomic>
#include <type_traits>

namespace fc {

constexpr uint32_t kPairChunkBytes = 32u * 128u;    // a chunk buffer: 32 rows of 128 bytes
constexpr uint32_t kPairLdsBytes = 160u * 1024u;
constexpr uint32_t pair_wave_bytes(int ring) { return (uint32_t)ring * kPairChunkBytes + 256u; }   // + a unit's list entries

constexpr uint32_t kPairRelu1 = 1, kPairRelu2 = 2, kPairCompactIn = 4, kPairCompactOut = 8, kPairBiasFirst1 = 16, kPairBiasFirst2 = 32;

struct PairArgs {
    int32_t x_rows, m;                  // rows of x, output positions
    int32_t c_in, c_mid, c_out;
    int32_t kch, ring;                  // 128-byte chunks of an input row, chunk buffers of a wave
    int32_t active, team;               // waves that own rows (the others load weights); log2 of those that share a unit's output channels
    int32_t mid_rows, out_rows;         // rows of the two weight matrices in LDS
    uint32_t flags;
};

// the lower halves of b <-> the upper halves of a
__device__ __forceinline__ void swap_halves(uint32_t &a, uint32_t &b)
{
    typedef uint32_t u32x2_sw __attribute__((ext_vector_type(2)));
    const u32x2_sw r = __builtin_bit_cast(u32x2_sw, __builtin_amdgcn_permlane32_swap(a, b, false, false));
    a = r.x;
    b = r.y;
}

// ---- what both kernels do with a wave's blocks of 32 channels x 32 rows: a lane holds four runs of four channels of one row ----

__device__ __forceinline__ void pair_start(f32x16_t &v, const float *bias, int block, int half, bool first)
{
    if (first) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 b = *reinterpret_cast<const float4 *>(bias + block * 32 + q * 8 + half * 4);
            v[q * 4] = b.x, v[q * 4 + 1] = b.y, v[q * 4 + 2] = b.z, v[q * 4 + 3] = b.w;
        }
    } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = 0.f;
    }
}

__device__ __forceinline__ void pair_finish(f32x16_t &v, const float *bias, int block, int half, bool first)
{
    if (first) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float4 b = *reinterpret_cast<const float4 *>(bias + block * 32 + q * 8 + half * 4);
        v[q * 4] += b.x, v[q * 4 + 1] += b.y, v[q * 4 + 2] += b.z, v[q * 4 + 3] += b.w;
    }
}

// N middle blocks -> the second layer's operands, rounded as the first layer's output is: two steps a block of a 16-bit type, one step of
// two blocks of bytes.  Channels past the last one become zeros: their weights are zeros, but zero times an infinite pixel is NaN, and NaN
// times the second layer's zeros would be every output channel's.  (c_mid is a multiple of 8: whole runs of both halves.  A branch that
// the whole wave takes, in the last blocks only.)
template <int DT, typename TO, int N>
__device__ __forceinline__ void pair_middle(f32x16_t *acc, const float *bias, int block0, int c_mid, int half, bool first, bool relu1, Frag<DT> *h)
{
    const bool past = (block0 + N) * 32 > c_mid;
#pragma unroll
    for (int b = 0; b < N; ++b) pair_finish(acc[b], bias, block0 + b, half, first);
    if constexpr (sizeof(TO) == 2) {
#pragma unroll
        for (int b = 0; b < N; ++b) {
            uint2 run[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                store4<DT, TO>(reinterpret_cast<TO *>(&run[q]), acc[b][q * 4], acc[b][q * 4 + 1], acc[b][q * 4 + 2], acc[b][q * 4 + 3]);
                if (relu1) run[q].x = relu_packed16(run[q].x), run[q].y = relu_packed16(run[q].y);
            }
            if (past) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if ((block0 + b) * 32 + q * 8 >= c_mid) run[q] = make_uint2(0u, 0u);
            }
#pragma unroll
            for (int q = 0; q < 4; q += 2) {
                swap_halves(run[q].x, run[q + 1].x);
                swap_halves(run[q].y, run[q + 1].y);
                h[b * 2 + (q >> 1)].v = make_uint4(run[q].x, run[q].y, run[q + 1].x, run[q + 1].y);
            }
        }
    } else {
        static_assert(N == 2, "a step of the 8-bit product");
        uint32_t run[2][4];
        auto pack = [&](auto relu) {
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    run[b][q] = pack4_e4m3<relu>(acc[b][q * 4], acc[b][q * 4 + 1], acc[b][q * 4 + 2], acc[b][q * 4 + 3]);
        };
        if (relu1) pack(std::true_type());
        else pack(std::false_type());
        if (past) {
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if ((block0 + b) * 32 + q * 8 >= c_mid) run[b][q] = 0u;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) swap_halves(run[0][q], run[1][q]);
        h[0].v = make_uint4(run[0][0], run[1][0], run[0][1], run[1][1]);
        h[0].v2 = make_uint4(run[0][2], run[1][2], run[0][3], run[1][3]);
    }
}

// N finished blocks, rounded, as blocks `at` .. at + N - 1 of a chunk in LDS (32 rows of 128 bytes, laid out like a gathered one)
template <int DT, typename TO, int N>
__device__ __forceinline__ void pair_pack(f32x16_t *acc, const float *bias, int block0, int lane, bool first, bool relu, unsigned char *stg, int at)
{
    const int l32 = lane & 31, half = lane >> 5;
    if constexpr (sizeof(TO) == 2) {
#pragma unroll
        for (int b = 0; b < N; ++b) {
            pair_finish(acc[b], bias, block0 + b, half, first);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                uint2 pk;
                store4<DT, TO>(reinterpret_cast<TO *>(&pk), acc[b][q * 4], acc[b][q * 4 + 1], acc[b][q * 4 + 2], acc[b][q * 4 + 3]);
                if (relu) pk.x = relu_packed16(pk.x), pk.y = relu_packed16(pk.y);
                *reinterpret_cast<uint2 *>(stg + (uint32_t)l32 * 128u + (uint32_t)(((at + b) * 4 + q) ^ FC_SWZ(l32)) * 16u + (uint32_t)half * 8u) = pk;
            }
        }
    } else {
        auto pack = [&](auto with_relu) {
#pragma unroll
            for (int b = 0; b < N; ++b) {
                pair_finish(acc[b], bias, block0 + b, half, first);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<uint32_t *>(stg + (uint32_t)l32 * 128u + (uint32_t)(((at + b) * 2 + (q >> 1)) ^ FC_SWZ(l32)) * 16u +
                                                  (uint32_t)((q & 1) * 8 + half * 4)) =
                        pack4_e4m3<with_relu>(acc[b][q * 4], acc[b][q * 4 + 1], acc[b][q * 4 + 2], acc[b][q * 4 + 3]);
            }
        };
        if (relu) pack(std::true_type());
        else pack(std::false_type());
    }
}

// N output blocks leave through LDS (4 KB of the wave's own) as whole lines: 8 lanes a row, row 8j + lane / 8 goes to to[j] (-1: nowhere)
template <int DT, typename TO, int N>
__device__ __forceinline__ void pair_store(f32x16_t *acc, const float *bias, int block0, int lane, bool first, bool relu2, unsigned char *stg,
                                           const int (&to)[4], int c_out, bool stream_out, TO *__restrict__ out)
{
    static_assert(N * (int)sizeof(TO) <= 4, "at most 128 bytes of a row");
    if (block0 * 32 >= c_out) return;
    pair_pack<DT, TO, N>(acc, bias, block0, lane, first, relu2, stg, 0);
    wave_lds_order();
    constexpr int per_row = N * 2 * (int)sizeof(TO);        // 16-byte pieces of a row
    const bool inside = (lane & 7) < per_row && block0 * 32 + (lane & 7) * (16 / (int)sizeof(TO)) < c_out;
    u32x4_t piece[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int row = j * 8 + (lane >> 3);
        piece[j] = *reinterpret_cast<const u32x4_t *>(stg + (uint32_t)row * 128u + (uint32_t)((lane & 7) ^ FC_SWZ(row)) * 16u);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        u32x4_t *at = reinterpret_cast<u32x4_t *>(out + (int64_t)(to[j] < 0 ? 0 : to[j]) * c_out + block0 * 32 + (lane & 7) * (16 / (int)sizeof(TO)));
        if (to[j] >= 0 && inside) {
            if (stream_out)
                __asm__ volatile("global_store_dwordx4 %0, %1, off nt" : : "v"(at), "v"(piece[j]) : "memory");
            else
                *at = piece[j];
        }
    }
    wave_lds_order();
}

template <int DT, typename TO, int NB, bool WIDE>
__global__ __launch_bounds__(sizeof(TO) == 1 ? 512 : 768, 1)
void k_conv_pair(PairArgs a, const int32_t *__restrict__ count, const int32_t *__restrict__ idx, const unsigned char *__restrict__ x,
                 const unsigned char *__restrict__ w1, const float *__restrict__ bias1, const unsigned char *__restrict__ w2,
                 const float *__restrict__ bias2, TO *__restrict__ out)
{
    static_assert(sizeof(TO) == (DT == FC_FP8 ? 1 : 2), "both layers store what they read");
    static_assert(WIDE || DT != FC_FP8, "a narrow middle: 16-bit storage");
    constexpr int ES = DT == FC_FP8 ? 1 : 2;
    constexpr uint32_t KSTEP = kStepBytes<DT>;
    constexpr int KK = 128 / (int)KSTEP;                // products of a chunk
    constexpr int MB = WIDE ? 2 : NB;                   // middle blocks made at a time
    constexpr int OB = WIDE ? NB : 2;                   // output blocks made at a time

    extern __shared__ __align__(16) unsigned char smem_raw[];
    const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>(smem_raw);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = (int)blockDim.x >> 6;
    const int l32 = lane & 31, half = lane >> 5;
    const int mid_chunks = (a.c_mid * ES + 127) >> 7;
    const uint32_t w1_bytes = (uint32_t)a.kch * (uint32_t)a.mid_rows * 128u, w2_bytes = (uint32_t)mid_chunks * (uint32_t)a.out_rows * 128u;
    const uint32_t bias_at = w1_bytes + w2_bytes;
    const int b1_room = (a.mid_rows + 63) & ~63;    // (a wave load brings 64 values; out_rows is a multiple of 64)
    const uint32_t waves_at = bias_at + (uint32_t)(b1_room + a.out_rows) * 4u;
    const unsigned char *const w1s = smem_raw, *const w2s = smem_raw + w1_bytes;
    const float *const b1s = reinterpret_cast<const float *>(smem_raw + bias_at), *const b2s = b1s + b1_room;
    const uint32_t my_at = waves_at + (uint32_t)wave * pair_wave_bytes(a.ring);
    unsigned char *const my = smem_raw + my_at;
    const uint32_t my0 = lds0 + my_at, idx0 = my0 + (uint32_t)a.ring * kPairChunkBytes;
    const int32_t *const idx_w = reinterpret_cast<const int32_t *>(my + (uint32_t)a.ring * kPairChunkBytes);

    const bool compact_in = (a.flags & kPairCompactIn) != 0, compact_out = (a.flags & kPairCompactOut) != 0;
    const bool first1 = (a.flags & kPairBiasFirst1) != 0, first2 = (a.flags & kPairBiasFirst2) != 0;
    const int rows = __builtin_amdgcn_readfirstlane(idx ? *count : a.m);
    const bool use_list = idx && !(compact_in && compact_out);      // (row j in, row j out: the list is not read)
    const bool stream_out = (int64_t)rows * a.c_out * (int)sizeof(TO) > (256ll << 20);     // (see k_conv_pw)

    // ---- the weights: rows of 128 bytes by chunk, their 16-byte pieces swizzled by the row; what lies past the last
    // channel on either side arrives as zeros.  Nobody waits for them before the first rows are on their way. ----
    const bool all_load = a.active == nw;
    const int loader = all_load ? wave : wave - a.active, loaders = all_load ? nw : nw - a.active;
    auto load_weights = [&](const unsigned char *w, int c_from, int c_to, int chunks, int rows_w, uint32_t at) {
        const u32x4_t rsrc = make_rsrc_words(w, (uint32_t)c_to * (uint32_t)c_from * (uint32_t)ES);
        const int pieces = (c_from * ES) >> 4;
        for (int ch = 0; ch < chunks; ++ch)
            for (int r0 = loader * 8; r0 < rows_w; r0 += loaders * 8) {
                const int row = r0 + (lane >> 3), piece = ch * 8 + ((lane & 7) ^ (int)FC_SWZ(row));
                const bool ok = row < c_to && piece < pieces;
                dma_load16(rsrc, ok ? (uint32_t)row * (uint32_t)c_from * (uint32_t)ES + (uint32_t)piece * 16u : kOutOfRange,
                           lds0 + at + ((uint32_t)ch * (uint32_t)rows_w + (uint32_t)r0) * 128u);
            }
    };
    if (loader >= 0) {
        load_weights(w1, a.c_in, a.c_mid, a.kch, a.mid_rows, 0u);
        load_weights(w2, a.c_mid, a.c_out, mid_chunks, a.out_rows, w1_bytes);
        const u32x4_t rsrc_1 = make_rsrc_words(bias1, bias1 ? (uint32_t)a.c_mid * 4u : 0u);
        const u32x4_t rsrc_2 = make_rsrc_words(bias2, bias2 ? (uint32_t)a.c_out * 4u : 0u);
        for (int i = loader * 64; i < b1_room; i += loaders * 64) dma_load4(rsrc_1, (uint32_t)(i + lane) * 4u, lds0 + bias_at + (uint32_t)i * 4u);
        for (int i = loader * 64; i < a.out_rows; i += loaders * 64)
            dma_load4(rsrc_2, (uint32_t)(i + lane) * 4u, lds0 + bias_at + (uint32_t)(b1_room + i) * 4u);
    }

    // ---- my share of the kept rows: units of 32, XCD j (workgroups b = j mod 8) takes the j-th contiguous eighth ----
    const int teams = a.active >> a.team, team = wave >> a.team, member = wave - (team << a.team);
    const int nwv = (int)gridDim.x * teams;
    const int wv = ((int)(blockIdx.x & 7) * ((int)gridDim.x >> 3) + (int)(blockIdx.x >> 3)) * teams + team;
    const int nb = (rows + 31) >> 5;
    const int share_q = nb / nwv, share_r = nb - share_q * nwv;
    const int b0 = wv * share_q + (wv * share_r) / nwv;
    const int nu = wave < a.active ? (wv + 1) * share_q + ((wv + 1) * share_r) / nwv - b0 : 0;

    const uint32_t row_bytes = (uint32_t)a.c_in * (uint32_t)ES;
    const u32x4_t rsrc_x = make_rsrc_words(x, (uint32_t)a.x_rows * row_bytes);
    const u32x4_t rsrc_i = make_rsrc_words(idx, (uint32_t)rows * 4u);
    // the last chunk of a row may be short: bit j says whether the piece this lane gathers in wave load j lies inside the row there
    const int tail8 = (int)(row_bytes >> 4) - (a.kch - 1) * 8;
    uint32_t tail_ok = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) tail_ok |= (uint32_t)(((lane & 7) ^ (int)FC_SWZ(j * 8 + (lane >> 3))) < tail8) << j;

    int issued = 0, mark_idx = 0;
    auto issue_idx = [&](int v) {
        if (!use_list) return;
        const uint32_t r = (uint32_t)(b0 + v) * 32u + (uint32_t)lane;
        lds_reads_done();
        dma_load4(rsrc_i, lane < 32 ? r * 4u : kOutOfRange, idx0);
        issued += 1;
        mark_idx = issued;
    };
    // a unit's rows: where row 8j + lane / 8 is stored (-1: no row) and the byte offset of the piece of it that this lane gathers
    int st_pr[2][4];
    uint32_t st_off[2][4];
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j) st_off[k][j] = kOutOfRange, st_pr[k][j] = -1;
    auto setup = [&](int v, int k) {
        const int r = (b0 + v) * 32 + l32;
        const bool valid = r < rows;
        int p = r;
        if (use_list) {
            wait_vmcnt_upto(issued - mark_idx);
            p = idx_w[l32];
        }
        const uint32_t off = valid ? (uint32_t)(compact_in ? r : p) * row_bytes : kOutOfRange;
        const int to = valid ? (compact_out ? r : p) : -1;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int row = j * 8 + (lane >> 3);
            const uint32_t o = (uint32_t)__shfl((int)off, row, 64);
            st_off[k][j] = o == kOutOfRange ? o : o + (uint32_t)((lane & 7) ^ FC_SWZ(row)) * 16u;
            st_pr[k][j] = __shfl(to, row, 64);
        }
    };
    // (all of this is the same for the whole wave; the compiler loses sight of that where the loops over chunks meet)
    // chunks sent for and not yet used up, the next one to send for (of unit u + ahead_unit) and its buffer
    int u = 0, ahead = 0, ahead_unit = 0, ahead_chunk = 0, ahead_buf = 0;
    auto send = [&]() {
        while (__builtin_amdgcn_readfirstlane(ahead) < a.ring) {
            ahead_chunk = __builtin_amdgcn_readfirstlane(ahead_chunk);
            ahead_unit = __builtin_amdgcn_readfirstlane(ahead_unit);
            ahead_buf = __builtin_amdgcn_readfirstlane(ahead_buf);
            if (ahead_chunk == a.kch) {
                if (ahead_unit == 1 || u + 1 >= nu) return;     // (two units' rows are held)
                setup(u + 1, 1);
                if (u + 2 < nu) issue_idx(u + 2);
                ahead_unit = 1;
                ahead_chunk = 0;
            }
            lds_reads_done();
            const bool last = ahead_chunk == a.kch - 1;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t o = ahead_unit ? st_off[1][j] : st_off[0][j];
                dma_load16_s(rsrc_x, last && !((tail_ok >> j) & 1u) ? kOutOfRange : o, (uint32_t)ahead_chunk * 128u,
                             my0 + (uint32_t)ahead_buf * kPairChunkBytes + (uint32_t)j * 1024u);
            }
            issued += 4;
            ++ahead;
            ++ahead_chunk;
            ahead_buf = ahead_buf + 1 == a.ring ? 0 : ahead_buf + 1;
        }
    };

    // lane reads row (lane & 31), in step kk the 16-byte piece 2 kk + half (8-bit storage: 4 kk + 2 half and the next)
    const uint32_t frag = (uint32_t)l32 * 128u + (uint32_t)((half * (int)(KSTEP / 32u)) ^ FC_SWZ(l32)) * 16u;

    const bool relu1 = (a.flags & kPairRelu1) != 0, relu2 = (a.flags & kPairRelu2) != 0;
    constexpr int SB = sizeof(TO) == 2 ? 2 : OB;        // output blocks stored together
    if (nu > 0) {
        issue_idx(0);
        setup(0, 0);
        if (nu > 1) issue_idx(1);
        send();
    }
    // (this wave's share of the weights was requested before everything counted in `issued`)
    wait_vmcnt_upto(issued);
    __syncthreads();

    // (narrow) the output blocks of this member of the team
    [[maybe_unused]] const int out_from = ((a.out_rows >> 6) * member >> a.team) * 2, out_to = ((a.out_rows >> 6) * (member + 1) >> a.team) * 2;
    int buf = 0;
    for (; u < nu; ++u) {
        const unsigned char *xs = my;
        Frag<DT> h[sizeof(TO) == 2 ? MB * 2 : 1];
        f32x16_t acc1[MB], acc2[OB];
        if constexpr (WIDE) {
            send();
            wait_vmcnt_upto(4 * (ahead - 1));
            xs = my + (uint32_t)buf * kPairChunkBytes;
            Frag<DT> xf[KK];
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) xf[kk].load(xs, frag ^ ((uint32_t)kk * KSTEP));
            --ahead;
#pragma unroll
            for (int b = 0; b < OB; ++b) pair_start(acc2[b], b2s, b, half, first2);
#pragma unroll 1
            for (int block = 0; block * 32 < a.c_mid; block += 2) {
#pragma unroll
                for (int b = 0; b < 2; ++b) pair_start(acc1[b], b1s, block + b, half, first1);
#pragma unroll
                for (int kk = 0; kk < KK; ++kk) {
                    if (DT == FC_FP8 && (uint32_t)kk * KSTEP >= row_bytes) break;      // (half a chunk: 64 channels)
                    Frag<DT> wf[2];
#pragma unroll
                    for (int b = 0; b < 2; ++b) wf[b].load(w1s + (block + b) * 4096, frag ^ ((uint32_t)kk * KSTEP));
#pragma unroll
                    for (int b = 0; b < 2; ++b) acc1[b] = mfma32<DT>(wf[b], xf[kk], acc1[b]);
                }
                pair_middle<DT, TO, 2>(acc1, b1s, block, a.c_mid, half, first1, relu1, h);
                // (the middle's chunk of these blocks, and the first step of it they are: bytes lie four blocks to a chunk)
                const unsigned char *ws = w2s + (uint32_t)(sizeof(TO) == 2 ? block >> 1 : block >> 2) * (uint32_t)a.out_rows * 128u;
                const int kk0 = sizeof(TO) == 2 ? 0 : (block >> 1) & 1;
#pragma unroll
                for (int kk = 0; kk < (sizeof(TO) == 2 ? KK : 1); ++kk) {
                    Frag<DT> wf[OB];
#pragma unroll
                    for (int b = 0; b < OB; ++b) wf[b].load(ws + b * 4096, frag ^ ((uint32_t)(kk0 + kk) * KSTEP));
#pragma unroll
                    for (int b = 0; b < OB; ++b) acc2[b] = mfma32<DT>(wf[b], h[kk], acc2[b]);
                }
            }
#pragma unroll
            for (int b = 0; b < OB; b += SB) pair_store<DT, TO, SB>(acc2 + b, b2s, b, lane, first2, relu2, my + (uint32_t)buf * kPairChunkBytes, st_pr[0], a.c_out, stream_out, out);
            buf = buf + 1 == a.ring ? 0 : buf + 1;
        } else {
#pragma unroll
            for (int b = 0; b < MB; ++b) pair_start(acc1[b], b1s, b, half, first1);
            for (int c = 0; c < a.kch; ++c) {
                send();
                wait_vmcnt_upto(4 * (ahead - 1));
                xs = my + (uint32_t)buf * kPairChunkBytes;
                const unsigned char *ws = w1s + (uint32_t)c * (uint32_t)a.mid_rows * 128u;
#pragma unroll
                for (int kk = 0; kk < KK; ++kk) {
                    Frag<DT> xf, wf[MB];
                    xf.load(xs, frag ^ ((uint32_t)kk * KSTEP));
#pragma unroll
                    for (int b = 0; b < MB; ++b) wf[b].load(ws + b * 4096, frag ^ ((uint32_t)kk * KSTEP));
#pragma unroll
                    for (int b = 0; b < MB; ++b) acc1[b] = mfma32<DT>(wf[b], xf, acc1[b]);
                }
                --ahead;
                buf = buf + 1 == a.ring ? 0 : buf + 1;
            }
            pair_middle<DT, TO, MB>(acc1, b1s, 0, a.c_mid, half, first1, relu1, h);
            unsigned char *const stg = const_cast<unsigned char *>(xs);
#pragma unroll 1
            for (int block = out_from; block < out_to; block += 2) {
#pragma unroll
                for (int b = 0; b < 2; ++b) pair_start(acc2[b], b2s, block + b, half, first2);
#pragma unroll
                for (int kk = 0; kk < 2 * MB; ++kk) {
                    Frag<DT> wf[2];
#pragma unroll
                    for (int b = 0; b < 2; ++b) wf[b].load(w2s + (uint32_t)(block + b) * 4096u, frag ^ ((uint32_t)kk * KSTEP));
#pragma unroll
                    for (int b = 0; b < 2; ++b) acc2[b] = mfma32<DT>(wf[b], h[kk], acc2[b]);
                }
                pair_store<DT, TO, 2>(acc2, b2s, block, lane, first2, relu2, stg, st_pr[0], a.c_out, stream_out, out);
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) st_off[0][j] = st_off[1][j], st_pr[0][j] = st_pr[1][j];
        ahead_unit = 0;     // (with two buffers and more the last chunk of a unit has sent for the next unit's first)
    }
}

// The same with more weights than LDS holds: they pass through it in stages of 128 bytes of the middle's channels, two
// buffers, sent for by the whole workgroup a stage ahead, a barrier a stage.  The input has 128 channels, the output 128 at most.  A wave owns
// one unit of 32 rows at a time, its pixels in registers for all stages (loaded in the product's lane order, which costs the address unit four times what whole lines do,
// but once a unit, all at once, and no LDS); a workgroup's units are dealt to its waves in as few passes as they need.
constexpr int kPairStreamWaves = 12;

template <int DT, typename TO>
__global__ __launch_bounds__(kPairStreamWaves * 64, 1)
void k_conv_pair_stream(PairArgs a, const int32_t *__restrict__ count, const int32_t *__restrict__ idx, const unsigned char *__restrict__ x,
                        const unsigned char *__restrict__ w1, const float *__restrict__ bias1, const unsigned char *__restrict__ w2,
                        const float *__restrict__ bias2, TO *__restrict__ out)
{
    constexpr int ES = DT == FC_FP8 ? 1 : 2;
    constexpr uint32_t KSTEP = kStepBytes<DT>;
    constexpr int KK = 128 / (int)KSTEP;
    constexpr int NW = kPairStreamWaves, NB = 4, KC = ES;    // output blocks, chunks of an input row: 128 channels either way
    constexpr int MID = 128 / ES;                       // channels of the middle a stage
    constexpr int MB = DT == FC_FP8 ? 2 : 1;            // middle blocks made at a time ...
    constexpr int STEPS = DT == FC_FP8 ? 1 : 2;         // ... and the steps of the second product that they are
    constexpr uint32_t W1_STAGE = (uint32_t)MID * KC * 128u, W2_STAGE = (uint32_t)NB * 32u * 128u, STAGE = W1_STAGE + W2_STAGE;

    extern __shared__ __align__(16) unsigned char smem_raw[];
    const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>(smem_raw);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    unsigned char *const stg = smem_raw + 2u * STAGE + (uint32_t)wave * kPairChunkBytes;
    float *const b1s = reinterpret_cast<float *>(smem_raw + 2u * STAGE + NW * kPairChunkBytes), *const b2s = b1s + a.c_mid;
    const bool compact_in = (a.flags & kPairCompactIn) != 0, compact_out = (a.flags & kPairCompactOut) != 0;
    const bool first1 = (a.flags & kPairBiasFirst1) != 0, first2 = (a.flags & kPairBiasFirst2) != 0;
    const uint32_t row_bytes = (uint32_t)a.c_in * (uint32_t)ES, mid_bytes = (uint32_t)a.c_mid * (uint32_t)ES;
    const int nstages = a.c_mid / MID;

    // one stage of weights into buffer `buf`: the middle's MID rows of w1, chunk by chunk, and 128 bytes of every row of w2
    const u32x4_t rsrc_1 = make_rsrc_words(w1, (uint32_t)a.c_mid * row_bytes), rsrc_2 = make_rsrc_words(w2, (uint32_t)a.c_out * mid_bytes);
    // (what a lane's part of a load adds to the stage's own offset does not change)
    constexpr int LOADS = (int)(STAGE / 1024u), MINE = (LOADS + NW - 1) / NW;
    uint32_t off[MINE];
#pragma unroll
    for (int k = 0; k < MINE; ++k) {
        const int i = k * NW + wave, j = i < (int)(W1_STAGE / 1024u) ? i : i - (int)(W1_STAGE / 1024u);
        const int row = (i < (int)(W1_STAGE / 1024u) ? j & (MID / 8 - 1) : j) * 8 + (lane >> 3);
        const uint32_t piece = (uint32_t)((lane & 7) ^ (int)FC_SWZ(row)) * 16u;
        off[k] = i < (int)(W1_STAGE / 1024u) ? (uint32_t)row * row_bytes + (uint32_t)(j / (MID / 8)) * 128u + piece
                                             : (row < a.c_out ? (uint32_t)row * mid_bytes + piece : kOutOfRange);
    }
    auto send = [&](int stage, int buf) {
        const uint32_t to = lds0 + (uint32_t)buf * STAGE;
        const uint32_t s1 = (uint32_t)(stage * MID) * row_bytes, s2 = (uint32_t)stage * 128u;
#pragma unroll
        for (int k = 0; k < MINE; ++k) {
            const int i = k * NW + wave;
            if (i < (int)(W1_STAGE / 1024u)) dma_load16_any(rsrc_1, off[k], s1, to + (uint32_t)i * 1024u);
            else if (i < LOADS) dma_load16_any(rsrc_2, off[k], s2, to + (uint32_t)i * 1024u);
        }
    };
    send(0, 0);
    for (int i = tid; i < a.c_mid; i += NW * 64) b1s[i] = bias1 ? bias1[i] : 0.f;
    for (int i = tid; i < NB * 32; i += NW * 64) b2s[i] = bias2 && i < a.c_out ? bias2[i] : 0.f;

    const int rows = __builtin_amdgcn_readfirstlane(idx ? *count : a.m);
    const bool use_list = idx && !(compact_in && compact_out);
    const bool stream_out = (int64_t)rows * a.c_out * (int)sizeof(TO) > (256ll << 20);
    const int units = (rows + 31) >> 5, grid = (int)gridDim.x;
    const int wg = (int)(blockIdx.x & 7) * (grid >> 3) + (int)(blockIdx.x >> 3);
    const int share_q = units / grid, share_r = units - share_q * grid;
    const int u0 = wg * share_q + wg * share_r / grid, nu = (wg + 1) * share_q + (wg + 1) * share_r / grid - u0;
    const int passes = (nu + NW - 1) / NW, per = passes ? (nu + passes - 1) / passes : 0;

    const uint32_t frag = (uint32_t)l32 * 128u + (uint32_t)((half * (int)(KSTEP / 32u)) ^ FC_SWZ(l32)) * 16u;
    int at = 0;     // stages so far
    for (int pass = 0; pass < passes; ++pass) {
        const int unit = pass * per + wave;
        const bool busy = wave < per && unit < nu;
        const int r = (u0 + unit) * 32 + l32;
        const bool valid = busy && r < rows;
        const int p = valid && use_list ? idx[r] : r;
        const int to = valid ? (compact_out ? r : p) : -1;
        Frag<DT> xf[KC * KK];
        f32x16_t acc2[NB];
        if (busy) {
            // (rows past the last one: some row's pixels, whose sums are not stored)
            const unsigned char *row = x + (size_t)(valid ? (compact_in ? r : p) : 0) * row_bytes + half * (KSTEP / 2);
#pragma unroll
            for (int kk = 0; kk < KC * KK; ++kk) xf[kk].load(row, (uint32_t)kk * KSTEP);
        }
        for (int stage = 0; stage < nstages; ++stage, ++at) {
            wait_vmcnt<0>();        // (this wave's part of the stage's weights)
            __syncthreads();
            if (stage + 1 < nstages || pass + 1 < passes) send(stage + 1 < nstages ? stage + 1 : 0, (at + 1) & 1);
            if (!busy) continue;
            const unsigned char *const w1s = smem_raw + (uint32_t)(at & 1) * STAGE, *const w2s = w1s + W1_STAGE;
            if (stage == 0) {
#pragma unroll
                for (int b = 0; b < NB; ++b) pair_start(acc2[b], b2s, b, half, first2);
            }
#pragma unroll
            for (int mb = 0; mb < MID / 32; mb += MB) {
                f32x16_t acc1[MB];
                Frag<DT> h[STEPS];
#pragma unroll
                for (int b = 0; b < MB; ++b) pair_start(acc1[b], b1s, stage * (MID / 32) + mb + b, half, first1);
#pragma unroll
                for (int c = 0; c < KC; ++c)
#pragma unroll
                    for (int kk = 0; kk < KK; ++kk) {
                        Frag<DT> wf[MB];
#pragma unroll
                        for (int b = 0; b < MB; ++b) wf[b].load(w1s + (c * MID + (mb + b) * 32) * 128, frag ^ ((uint32_t)kk * KSTEP));
#pragma unroll
                        for (int b = 0; b < MB; ++b) acc1[b] = mfma32<DT>(wf[b], xf[c * KK + kk], acc1[b]);
                    }
                pair_middle<DT, TO, MB>(acc1, b1s, stage * (MID / 32) + mb, INT32_MAX, half, first1, (a.flags & kPairRelu1) != 0, h);
#pragma unroll
                for (int kk = 0; kk < STEPS; ++kk) {
                    const int step = DT == FC_FP8 ? mb / 2 : mb * 2 + kk;
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        Frag<DT> wf;
                        wf.load(w2s + b * 4096, frag ^ ((uint32_t)step * KSTEP));
                        acc2[b] = mfma32<DT>(wf, h[kk], acc2[b]);
                    }
                }
            }
        }
        if (!busy) continue;
        int st_pr[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) st_pr[j] = __shfl(to, j * 8 + (lane >> 3), 64);
        constexpr int SB = sizeof(TO) == 2 ? 2 : 4;
#pragma unroll
        for (int b = 0; b < NB; b += SB)
            pair_store<DT, TO, SB>(acc2 + b, b2s, b, lane, first2, (a.flags & kPairRelu2) != 0, stg, st_pr, a.c_out, stream_out, out);
    }
}

// ---------------------------------------------------------------------------

namespace {

struct PairCut {
    bool wide, stream;      // a wide middle; weights that pass through LDS
    int blocks;             // NB
    int waves, ring;
    PairArgs a;
    uint32_t lds;
};

// How the pair is cut, false if it does not fit: both layers' weights in LDS and two chunk buffers each for eight waves at least where the
// middle is wide, four where it is narrow.  (Or, with a wide middle, the weights pass through LDS: see pair_stream_cut.)
bool pair_resident_cut(const Geom &g1, const Geom &g2, int dtype, PairCut *cut)
{
    const int es = dtype == FC_FP8 ? 1 : 2;
    PairCut c = {};
    PairArgs &a = c.a;
    a.m = g1.m;
    a.x_rows = (g1.flags & FC_COMPACT_IN) ? g1.m : g1.n * g1.h * g1.w;
    a.c_in = g1.c_in, a.c_mid = g1.c_out, a.c_out = g2.c_out;
    a.kch = (a.c_in * es + 127) / 128;
    a.flags = (g1.flags & FC_RELU ? kPairRelu1 : 0) | (g2.flags & FC_RELU ? kPairRelu2 : 0) |
              (g1.flags & FC_COMPACT_IN ? kPairCompactIn : 0) | (g2.flags & FC_COMPACT_OUT ? kPairCompactOut : 0);
    c.wide = a.kch == 1 && a.c_out <= (dtype == FC_FP8 ? 128 : 64) && a.c_mid > 64;
    if (c.wide) {
        c.blocks = a.c_out <= 64 ? 2 : 4;
        a.mid_rows = (a.c_mid + 63) & ~63;
        a.out_rows = c.blocks * 32;
    } else {
        if (dtype == FC_FP8 || a.c_mid > 64) return false;
        c.blocks = a.c_mid <= 32 ? 1 : 2;
        a.mid_rows = c.blocks * 32;
        a.out_rows = (a.c_out + 63) & ~63;
    }
    const int mid_chunks = (a.c_mid * es + 127) / 128;
    const uint32_t fixed = ((uint32_t)a.kch * a.mid_rows + (uint32_t)mid_chunks * a.out_rows) * 128u +
                           (uint32_t)(((a.mid_rows + 63) & ~63) + a.out_rows) * 4u;
    if (fixed >= kPairLdsBytes) return false;
    const uint32_t room = kPairLdsBytes - fixed;
    // A wave with rows for every unit of a CU, the rest of LDS for the chunks on their way; where that leaves waves idle, several share a
    // unit's output channels (each makes the whole middle).  Eight waves at least fetch the weights.
    const int units = (g1.m + 31) / 32, per_cu = (units + conv_grid_cus() - 1) / conv_grid_cus();
    const int fit = (int)(room / pair_wave_bytes(2)), most = dtype == FC_FP8 ? 8 : 12;
    if (fit < (c.wide ? 8 : 4)) return false;
    a.team = 0;
    if (!c.wide)
        while (a.team < 2 && per_cu << (a.team + 1) <= std::min(fit, 8) && 64 << (a.team + 1) <= a.out_rows) ++a.team;
    a.active = std::min({per_cu, fit >> a.team, most >> a.team}) << a.team;
    c.waves = std::max(8, a.active);
    c.ring = std::min(std::max(2, a.kch + 1), (int)((room / (uint32_t)a.active - 256u) / kPairChunkBytes));
    a.ring = c.ring;
    c.lds = fixed + (uint32_t)a.active * pair_wave_bytes(c.ring);
    *cut = c;
    return true;
}

bool pair_stream_cut(const Geom &g1, const Geom &g2, int dtype, PairCut *cut)
{
    const int es = dtype == FC_FP8 ? 1 : 2;
    PairCut c = {};
    c.wide = c.stream = true;
    PairArgs &a = c.a;
    a.m = g1.m;
    a.c_in = g1.c_in, a.c_mid = g1.c_out, a.c_out = g2.c_out;
    a.flags = (g1.flags & FC_RELU ? kPairRelu1 : 0) | (g2.flags & FC_RELU ? kPairRelu2 : 0) |
              (g1.flags & FC_COMPACT_IN ? kPairCompactIn : 0) | (g2.flags & FC_COMPACT_OUT ? kPairCompactOut : 0);
    if (a.c_in != 128 || (a.c_mid * es) % 128 != 0 || a.c_out > 128 || a.c_mid < a.c_out) return false;
    // With few units a CU the weights are too much to fetch for them.  128 -> 512 -> 128, half kept, chained and without a mask, us, two launches -> one: bf16 on 4 x 40 x 40
    // 12.2 -> 14.7, 13.3 -> 14.8, on 8 x 40 x 40 14.6 -> 14.9, 15.5 -> 15.5, on 12 x 50 x 50 17.2 -> 15.9, 21.3 -> 17.4, on 32 x 60 x 80 54.6 -> 28.1, 95.6 -> 49.7; E4M3 on 8 x 40 x 40
    // 13.4 -> 13.3, 14.7 -> 14.0, on 12 x 50 x 50 15.3 -> 14.1, 17.9 -> 14.6, on 32 x 60 x 80 31.1 -> 23.1, 46.0 -> 37.9.  (Three such pairs of a ResNet-50 stage; the next
    // stage's 256 -> 1024 -> 256 are too many sums for three waves a SIMD: on 32 x 30 x 40 44 us as two, 49 .. 61 with one wave a SIMD, 46 with
    // two waves a unit.)
    if (a.m < 24000) return false;
    c.waves = kPairStreamWaves;
    c.lds = 2u * (uint32_t)(128 * 128 + 128 * 128) + (uint32_t)c.waves * kPairChunkBytes + (uint32_t)(a.c_mid + 128) * 4u;
    if (c.lds > kPairLdsBytes) return false;
    *cut = c;
    return true;
}

bool pair_cut(const Geom &g1, const Geom &g2, int dtype, PairCut *cut)
{
    return pair_resident_cut(g1, g2, dtype, cut) || pair_stream_cut(g1, g2, dtype, cut);
}

template <typename TO>
using PairKernel = void (*)(PairArgs, const int32_t *, const int32_t *, const unsigned char *, const unsigned char *, const float *,
                            const unsigned char *, const float *, TO *);

template <typename TO, PairKernel<TO> KERN>
hipError_t launch_pair(const PairCut &c, const void *x, const void *w1, const float *bias1, const void *w2, const float *bias2,
                       const int32_t *idx, const int32_t *count, void *out, hipStream_t s)
{
    PairKernel<TO> kern = KERN;
    // the dynamic LDS limit is raised once per function and device
    static std::atomic<uint64_t> attr_devices{0};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t dev_bit = 1ull << (dev & 63);
    if (!(attr_devices.load(std::memory_order_acquire) & dev_bit)) {
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kPairLdsBytes);
        if (e != hipSuccess) return e;
        attr_devices.fetch_or(dev_bit, std::memory_order_release);
    }
    hipLaunchKernelGGL(kern, dim3(conv_grid_cus()), dim3(c.waves * 64), c.lds, s, c.a, count, idx, (const unsigned char *)x,
                       (const unsigned char *)w1, bias1, (const unsigned char *)w2, bias2, (TO *)out);
    return hipGetLastError();
}

} // namespace

bool conv_pair_supported(const Geom &g1, const Geom &g2, int dtype)
{
    if (dtype != FC_BF16 && dtype != FC_F16 && dtype != FC_FP8) return false;
    const int unit = dtype == FC_FP8 ? 16 : 8;
    for (const Geom *g : {&g1, &g2}) {
        if (!(g->kh == 1 && g->kw == 1 && g->sh == 1 && g->sw == 1 && g->ph == 0 && g->pw == 0)) return false;
        if (g->c_in % unit != 0 || g->c_out % unit != 0) return false;
        if ((uint64_t)g->n * g->h * g->w * g->c_in * (dtype == FC_FP8 ? 1u : 2u) >= kBufferLimit) return false;
    }
    if (g1.n != g2.n || g1.h != g2.h || g1.w != g2.w || g1.c_out != g2.c_in || (uint64_t)g1.m * 4u >= kBufferLimit) return false;
    PairCut c;
    return pair_cut(g1, g2, dtype, &c);
}

hipError_t launch_conv_pair(const Geom &g1, const Geom &g2, int dtype, bool bias_first1, bool bias_first2, const void *x, const void *w1,
                            const float *bias1, const void *w2, const float *bias2, const int32_t *idx, const int32_t *count, void *out,
                            hipStream_t s)
{
    PairCut c;
    if (!pair_cut(g1, g2, dtype, &c)) return hipErrorInvalidValue;
    c.a.flags |= (bias_first1 ? kPairBiasFirst1 : 0) | (bias_first2 ? kPairBiasFirst2 : 0);
#define FC_PAIR_CALL(TO, ...) launch_pair<TO, __VA_ARGS__>(c, x, w1, bias1, w2, bias2, idx, count, out, s)
    if (c.stream) {
        if (dtype == FC_FP8) return FC_PAIR_CALL(uint8_t, k_conv_pair_stream<FC_FP8, uint8_t>);
        return dtype == FC_BF16 ? FC_PAIR_CALL(uint16_t, k_conv_pair_stream<FC_BF16, uint16_t>) : FC_PAIR_CALL(uint16_t, k_conv_pair_stream<FC_F16, uint16_t>);
    }
    if (dtype == FC_FP8)
        return c.blocks == 2 ? FC_PAIR_CALL(uint8_t, k_conv_pair<FC_FP8, uint8_t, 2, true>) : FC_PAIR_CALL(uint8_t, k_conv_pair<FC_FP8, uint8_t, 4, true>);
    if (dtype == FC_BF16)
        return c.wide ? FC_PAIR_CALL(uint16_t, k_conv_pair<FC_BF16, uint16_t, 2, true>)
                      : (c.blocks == 1 ? FC_PAIR_CALL(uint16_t, k_conv_pair<FC_BF16, uint16_t, 1, false>) : FC_PAIR_CALL(uint16_t, k_conv_pair<FC_BF16, uint16_t, 2, false>));
    return c.wide ? FC_PAIR_CALL(uint16_t, k_conv_pair<FC_F16, uint16_t, 2, true>)
                  : (c.blocks == 1 ? FC_PAIR_CALL(uint16_t, k_conv_pair<FC_F16, uint16_t, 1, false>) : FC_PAIR_CALL(uint16_t, k_conv_pair<FC_F16, uint16_t, 2, false>));
#undef FC_PAIR_CALL
}

} // namespace fc
