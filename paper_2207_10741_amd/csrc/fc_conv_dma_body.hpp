// The body of the tiled kernel (see fc_conv_mfma.hip), included in its two homes, k_conv_dma and conv_list_tiles.  (As an inlined function in both, k_conv_dma is scheduled and allocated otherwise: 512 -> 512 on 32 x 15 x 20,
// half kept, 39.7 -> 41.2 us, E4M3 23.6 -> 24.7.)
    constexpr int NT = WM * WN * 64;
    constexpr int RPP = NT / 8;        // rows covered by one pass of wave loads
    constexpr int XR = TM / RPP;       // wave loads per thread for the activation tile
    constexpr int WR = TN / RPP;       // ... for the weight tile
    constexpr int L = XR + WR;         // loads per thread per stage
    constexpr int WTM = TM / WM, WTN = TN / WN;
    constexpr int PB = WTM / 32, CB = WTN / 32;
    constexpr int ES = DT == FC_FP8 ? 1 : 2;               // bytes per stored element
    constexpr int TK = kStageBytes / ES;                   // reduction elements per stage
    constexpr int EPP = 16 / ES;                           // elements per 16-byte piece
    constexpr uint32_t KSTEP = kStepBytes<DT>;             // bytes of a row per matrix instruction
    constexpr int KK = kStageBytes / (int)KSTEP;           // matrix instructions per stage and block pair
    constexpr int ODT = DT == FC_FP8 ? FC_BF16 : DT;       // 16-bit output format
    // register sets of operand fragments: the 16-bit types fetch step kk + 1 while step kk is
    // multiplied; fp8 fragments are twice as large and its instructions twice as long, so one set,
    // refilled behind the multiplies of a step, keeps the kernel inside the register file
    constexpr int FB = (DT == FC_FP8 && TM * TN >= 128 * 128) ? 1 : 2;
    constexpr int PAIR_IT = (TM * TAPC + NT - 1) / NT;
    constexpr int PAIR_CH = PAIR_IT < 5 ? PAIR_IT : 5;
    constexpr int STAGE_BYTES = (TM + TN) * 128;
    static_assert(TM % RPP == 0 && TN % RPP == 0 && WTM % 32 == 0 && WTN % 32 == 0, "tile shape");
    static_assert(TM <= NT && TN <= NT, "set-up assumes one thread per row / channel");
    static_assert(NB >= 2 && (NB - 1) * L <= 63, "vmcnt is a 6-bit counter");
    constexpr bool HALO = SL > 0;
    constexpr size_t REGION = dma_stage_region_bytes<TM, TN, NB, SL, NBW>();
    static_assert(!HALO || (TAPC == 9 && SL % RPP == 0 && SL <= NT && SL > TM && (NBW == 2 || NBW == 3)),
                  "shared-halo loop: 3x3 kernels, whole load passes, one thread per slot");

    extern __shared__ __align__(16) unsigned char smem_raw[];
    unsigned char *stage0 = smem_raw;                                   // [NB][TM + TN][128]
    int32_t *row_p = reinterpret_cast<int32_t *>(smem_raw + REGION);
    int32_t *row_base = row_p + TM;
    int32_t *row_img = row_base + TM;
    int32_t *row_hw = row_img + TM;
    uint32_t *row_bits = reinterpret_cast<uint32_t *>(row_hw + TM);
    // shared-halo loop only: centre slot of every row, and per slot the pixel of kernel row 0,
    // its packed (ih, iw) and one "inside the image and relevant" bit per kernel row
    int32_t *row_cs = reinterpret_cast<int32_t *>(row_bits + TM);
    int32_t *slot_pix = row_cs + TM;
    int32_t *slot_hw = slot_pix + SL;
    uint32_t *slot_bits = reinterpret_cast<uint32_t *>(slot_hw + SL);
    int32_t *scan_part = reinterpret_cast<int32_t *>(slot_bits + SL);
    const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>(smem_raw); // LDS byte address of the stage buffers

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wave_m = wave % WM, wave_n = wave / WM;
    const int slot = tid & 7, prow = tid >> 3;

    // Kept rows.  With a list they are given.  Without one but with a mask (the launcher does
    // this only for layers of at most 16 positions per thread) the workgroup ranks the kept
    // positions itself: thread t labels positions 16t .. 16t+15 (centre tap, Sec. III-B) and a
    // prefix sum over the workgroup gives the rank of its first kept position; the set-up of a
    // tile then has every thread drop its positions of that tile's rank range into row_p.  A
    // small layer so needs no compaction launch before this one.
    const bool packed_masks = (g.flags & FC_PACKED_MASKS) != 0; // masks are one bit per pixel
    const bool inline_rank = !OWN && !LIST && !idx && mask_in;
    uint32_t rank_flags = 0;
    int rank_base = 0;
    int rows = g.m;
    if (inline_rank) {
        MaskGeom mg = mask_geom(g.n, g.h, g.w, g.kh, g.kw, g.sh, g.sw, g.ph, g.pw, g.dh, g.dw, g.ho, g.wo);
        mg.packed_in = (g.flags & FC_PACKED_MASKS) ? 1 : 0;
        if (!mg.packed_in && (reinterpret_cast<uintptr_t>(mask_in) & 15u)) mg.identity = 0; // the 128-bit path needs alignment
        rank_flags = kept_flags16(mg, mask_in, (int64_t)tid * 16);
        const int cnt = __popc(rank_flags);
        const int incl = wave_inclusive_scan(cnt);
        if (lane == 63) row_p[wave] = incl;
        __syncthreads();
        int before = 0, total = 0;
#pragma unroll
        for (int v = 0; v < NT / 64; ++v) {
            const int t = row_p[v];
            before += v < wave ? t : 0;
            total += t;
        }
        rank_base = before + incl - cnt;
        rows = total;
        __syncthreads(); // row_p is free again
    } else if (LIST) {
        rows = list_rows;
    } else if (!OWN && idx) {
        rows = *count;
    }
    const int n_nt = (g.c_out + TN - 1) / TN;
    const int ntiles = ((rows + TM - 1) / TM) * n_nt;
    const int taps = TAPC == 32 ? g.kh * g.kw : TAPC;
    const int kwid = TAPC == 32 ? g.kw : (TAPC == 9 ? 3 : 1);
    const int cchunks = (g.c_in + TK - 1) / TK;
    const int tap_pieces = g.c_in / EPP; // PACK: a tap's 16-byte pieces
    const int stages = PACK ? (taps * tap_pieces + 7) >> 3 : taps * cchunks;
    const bool self_tap = TAPC == 1 && g.ph == 0 && g.pw == 0;
    const u32x4_t rsrc_x = make_rsrc_words(x, (uint32_t)g.n * g.h * g.w * g.c_in * (uint32_t)ES);
    const u32x4_t rsrc_w = make_rsrc_words(w, (uint32_t)g.c_out * taps * g.c_in * (uint32_t)ES);

    // fragment addressing: lane reads row (lane & 31) of a 32-row block; in step kk that is
    // the 16-byte piece 2*kk + (lane >> 5) (fp8: the pieces 4*kk + 2*(lane >> 5) and the one
    // after it), stored at slot piece ^ ((row >> 1) & 7); all block bases are multiples of 32
    // rows, so the swizzle term depends on the lane only
    constexpr uint32_t HALF = KSTEP / 32u; // piece index of the upper half-wave within a step
    const uint32_t frag_row = (uint32_t)(lane & 31) * 128u;
    const uint32_t frag_t16 = (uint32_t)(((lane >> 5) * HALF) ^ FC_SWZ(lane & 31)) * 16u;

    // Tile order.  Workgroups are dispatched round-robin over the 8 XCDs, each with its own L2, so XCD j takes the
    // j-th contiguous eighth of the order: its tiles share neighbouring image rows (the halo of the 3x3 taps) in
    // that L2.  The order is by groups of `1 << nt_log` channel tiles, within a group row tile by row tile: the
    // pixels of a row tile are read by one XCD per group, a group's weights by the XCDs that share it.  Against one
    // channel tile after another (half kept, chained): 256 -> 256 stride 2 from 32 x 60 x 80 reads 174 -> 68 MB past the L2s, 48.8 -> 43.2 us;
    // 1024 -> 512 on 32 x 30 x 40 167 -> 54 MB, 40.7 -> 36.8; 1024 -> 256 there 83 -> 46 MB, 25.2 -> 23.4; 512 -> 512 3x3 on 32 x 15 x 20
    // 94 -> 30 MB, over six masks each that keep 0.3 / 0.5 / 0.7 34.2 / 43.3 / 43.6 -> 33.7 / 42.3 / 42.8 (one mask by itself 39 to 46 either way: it decides which CUs
    // get two tiles that go tap by tap).  What it costs shows where pixels and weights fit an L2 anyhow: 256 -> 256 on 8 x 30 x 40 16.8 -> 17.0, 128 -> 128 on
    // 8 x 60 x 80 14.7 -> 15.0.
    const int n_mt = (rows + TM - 1) / TM;
    int nt_log = 0;
    {
        // doubling a group halves the readers of the pixels and doubles those of the weights (both in units of c_in)
        const float px = (float)rows * (float)(taps == 1 ? 1 : g.sh * g.sw) * (float)(n_nt * n_nt);
        const float wt = 16.f * (float)g.c_out * (float)taps;
        while (!(n_nt & ((2 << nt_log) - 1)) && px > wt * (float)(1 << (2 * nt_log))) ++nt_log;
    }
    // Split-K: when there are fewer tiles than workgroups (small layers, or few kept rows)
    // the reduction of every tile is cut into S equal runs of stages, one work unit each, so
    // that the serial K loop of a workgroup gets S times shorter and the chip fills up.
    // Units of one tile are adjacent in the order, so they share an XCD.  S is the same in
    // every workgroup (it depends on the kept count and the grid only).
    int S = 1;
    if (!OWN && partials && ntiles > 0) S = split_k_splits(ntiles, (int)gridDim.x, HALO ? g.kh * cchunks : stages, stages, (g.flags & kOneUnitPerCu) != 0);
    const int nunits = ntiles * S;
    const int per_xcd = (nunits + 7) >> 3;
    const int xcd = blockIdx.x & 7;

    // ---- zero-fill of the irrelevant output rows (none for the dense layer) ----
    // The grid is sized for the dense row count, so with a kept share r about 1 - r of
    // the workgroups have no tile: when there are enough of them they alone clear the
    // irrelevant rows (about one tile's worth of rows each, off the critical path of the
    // tiles); otherwise every workgroup clears its share before its tiles.  A wave looks
    // at 64 positions at a time and stores whole 16-byte pieces with all lanes.
    if (!OWN && mask_in && !(g.flags & FC_SKIP_ZERO_FILL)) {
        const int slots = gridDim.x >> 3;
        const int idle_slots = slots > per_xcd ? slots - per_xcd : 0;
        const bool idle_only = idle_slots > 0 && idle_slots * 8 >= (int)(gridDim.x >> 4);
        const int my_slot = blockIdx.x >> 3;
        if (!idle_only || my_slot >= per_xcd) {
            const int nworkers = (idle_only ? idle_slots * 8 : (int)gridDim.x) * (NT / 64);
            const int worker = (idle_only ? (my_slot - per_xcd) * 8 + xcd : (int)blockIdx.x) * (NT / 64) + wave;
            int32_t *dropped = reinterpret_cast<int32_t *>(smem_raw) + wave * 64; // per-wave list
            const int cpr = g.c_out * (int)sizeof(TO) / 16; // 16-byte pieces per row
            u32x4_t *o4 = reinterpret_cast<u32x4_t *>(out);
            const u32x4_t zero4 = {0u, 0u, 0u, 0u};
            const int ch0 = -g.ph + g.dh * ((g.kh - 1) / 2), cw0 = -g.pw + g.dw * ((g.kw - 1) / 2);
            // Where there are more waves than blocks of 64 positions, as many as have a row's sixteen pieces each share a block: one wave alone
            // stores 1 KB at a time, and 512 -> 2048 on 2 x 7 x 7 has two blocks of 128 KB to clear (15.2 -> 6.2 us, chained 6.1; 320 -> 1280 on 32 x 7 x 7
            // 12.3 -> 6.7, 256 -> 1024 on 2 x 14 x 14 11.7 -> 5.2).  Narrow rows leave one wave little, and more of them disturb the tiles (960 -> 160 on
            // 32 x 14 x 14 shared by all 10.3 -> 10.6).
            const int nblocks = (g.m + 63) >> 6, parts = max(min(nworkers / nblocks, cpr / 16), 1);
            for (int item = worker; item < nblocks * parts; item += nworkers) {
                const int blk = item / parts, part = item - blk * parts;
                const int pp = blk * 64 + lane;
                bool kept = true;
                if (pp < g.m) {
                    if (mask_out) {
                        kept = mask_at(mask_out, pp, packed_masks);
                    } else {
                        const int q = (int)fast_div((uint32_t)pp, g.div_wo), ow = pp - q * g.wo;
                        const int b = (int)fast_div((uint32_t)q, g.div_ho), oh = q - b * g.ho;
                        const int ih = min(max(oh * g.sh + ch0, 0), g.h - 1);
                        const int iw = min(max(ow * g.sw + cw0, 0), g.w - 1);
                        kept = mask_at(mask_in, (int64_t)(b * g.h + ih) * g.w + iw, packed_masks);
                    }
                }
                const uint64_t drop = __ballot(!kept);
                const int nd = __popcll(drop);
                if (!kept) dropped[__popcll(drop & ((1ull << lane) - 1ull))] = pp; // in position order
                wave_lds_order();
                const int total = nd * cpr;
                for (int c = part * 64 + lane; c < total; c += parts * 64) {
                    const int rk = c / cpr, pc = c - rk * cpr;
                    __builtin_nontemporal_store(zero4, o4 + (int64_t)dropped[rk] * cpr + pc);
                }
                wave_lds_order();
            }
        }
    }
    for (int slot_t = blockIdx.x >> 3; slot_t < per_xcd; slot_t += gridDim.x >> 3) {
        const int unit = xcd * per_xcd + slot_t;
        if (unit >= nunits) break;
        const int tile = unit / S, split = unit - tile * S;
        // (32-bit divisions only, and positions through multiplies: the 64-bit ones were a third of the
        // 4 300 cycles a workgroup took to its rows' addresses)
        int s_begin = 0, s_end = stages;
        if (S > 1) {
            s_begin = (int)((uint32_t)(split * stages) / (uint32_t)S);
            s_end = (int)((uint32_t)((split + 1) * stages) / (uint32_t)S);
        }
        int nst = s_end - s_begin; // stages of this unit
        const int grp = tile / (n_mt << nt_log), in_grp = tile - grp * (n_mt << nt_log);
        const int mt = in_grp >> nt_log, nt = (grp << nt_log) + (in_grp & ((1 << nt_log) - 1));
        const int co0 = nt * TN;

        __syncthreads(); // the previous tile's epilogue is done with LDS
        if (inline_rank) {
            // every thread drops its kept positions whose rank falls into this tile
            if (tid < TM) row_p[tid] = -1;
            __syncthreads();
            const int lo = mt * TM;
            int r = rank_base;
            uint32_t f = rank_flags;
            if (r < lo + TM && r + __popc(f) > lo) {
                while (f) {
                    const int j = __ffs((int)f) - 1;
                    f &= f - 1;
                    if (r >= lo && r < lo + TM) row_p[r - lo] = tid * 16 + j;
                    ++r;
                }
            }
            __syncthreads();
        }
        bool dropped_row = false; // OWN: this thread's row is an irrelevant position
        int sa_p = -1, sa_ow = 0, sa_ih0 = 0, sa_iw0 = 0, sa_b = 0; // this thread's row (tid < TM)
        if (tid < TM) {
            const int m = mt * TM + tid;
            int p = -1, base = 0, b = 0, hw = 0;
            if (m < rows) {
                p = inline_rank ? row_p[tid] : (LIST || (!OWN && idx) ? idx[m] : m);
                if constexpr (OWN) dropped_row = !position_kept(g, mask_in, mask_out, m);
                const int q = (int)fast_div((uint32_t)p, g.div_wo), ow = p - q * g.wo;
                b = (int)fast_div((uint32_t)q, g.div_ho);
                const int oh = q - b * g.ho;
                const int ih0 = oh * g.sh - g.ph, iw0 = ow * g.sw - g.pw;
                sa_p = p; sa_ow = ow; sa_ih0 = ih0; sa_iw0 = iw0; sa_b = b;
                base = (b * g.h + ih0) * g.w + iw0;
                // compacted input (1x1, unit stride, no padding): the row's pixel is row m of x
                if constexpr (CMP) {
                    if (g.flags & FC_COMPACT_IN) base = m;
                }
                hw = (int)(((uint32_t)ih0 & 0xffffu) | ((uint32_t)iw0 << 16));
            }
            row_p[tid] = p;
            row_base[tid] = base;
            row_img[tid] = b;
            row_hw[tid] = hw;
            // an unpadded 1x1 kernel reads exactly the pixel that decided to keep the position:
            // inside the image and relevant by construction, nothing to look up
            row_bits[tid] = (self_tap && p >= 0) ? 1u : 0u;
        }
        // The accumulators start from the bias (in the first K-split only), so the epilogue has
        // nothing to add: every lane fetches the bias of its own channels now and the loads
        // are long back when the set-up is done.
        float4 bias_q[CB][4];
#pragma unroll
        for (int b = 0; b < CB; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int co = co0 + wave_n * WTN + b * 32 + q * 8 + (lane >> 5) * 4;
                bias_q[b][q] = (bias && split == 0 && co < g.c_out) ? *reinterpret_cast<const float4 *>(bias + co)
                                                                    : make_float4(0.f, 0.f, 0.f, 0.f);
            }
        __syncthreads();
        bool use_halo = false;
        int ns = 0; // slots on this tile's pixel line
        if constexpr (HALO) {
            int cnt = 0, lead = 0;
            bool ladj = false, radj = false;
            if (tid < TM) {
                cnt = 1;
                if (sa_p >= 0) {
                    ladj = tid > 0 && row_p[tid - 1] == sa_p - 1 && sa_ow > 0;
                    radj = tid < TM - 1 && row_p[tid + 1] == sa_p + 1 && sa_ow < g.wo - 1;
                    lead = ladj ? 0 : 1;
                    cnt = 1 + lead + (radj ? 0 : 1);
                }
            }
            const int incl = wave_inclusive_scan(cnt);
            if (lane == 63) scan_part[wave] = incl;
            if (tid < SL) slot_bits[tid] = 0;
            __syncthreads();
            int before = 0;
#pragma unroll
            for (int v = 0; v < NT / 64; ++v) {
                const int t = scan_part[v];
                before += v < wave ? t : 0;
                ns += t;
            }
            // (one slot to spare: a row past the end of the list still reads "its" three slots)
            use_halo = ns + 1 <= SL;
            if (use_halo && tid < TM) {
                const int cs = before + incl - cnt + lead;
                row_cs[tid] = cs;
                if (sa_p >= 0) {
                    const int iwc = sa_iw0 + 1; // kw = 1, unit dilation
                    const int pixc = (sa_b * g.h + sa_ih0) * g.w + iwc;
                    const int ih16 = (int)((uint32_t)sa_ih0 & 0xffffu);
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
            if (use_halo) {
                // one thread per (slot, kernel row): inside the image and relevant?
                constexpr int SIT = (SL * 3 + NT - 1) / NT;
                int ssl_[SIT], skh_[SIT], spix_[SIT];
                bool sin_[SIT];
#pragma unroll
                for (int i = 0; i < SIT; ++i) {
                    const int pair = tid + i * NT;
                    const int sl = pair / 3, kh_i = pair - sl * 3;
                    const bool live = sl < ns;
                    const int s2 = live ? sl : 0;
                    const int hw = slot_hw[s2];
                    const int ih = (int)(int16_t)(hw & 0xffff) + kh_i * g.dh;
                    const int iw = hw >> 16;
                    const bool inb = live && ih >= 0 && ih < g.h && iw >= 0 && iw < g.w;
                    ssl_[i] = s2;
                    skh_[i] = kh_i;
                    sin_[i] = inb;
                    spix_[i] = inb ? slot_pix[s2] + kh_i * g.dh * g.w : 0;
                }
                uint32_t smv[SIT];
#pragma unroll
                for (int i = 0; i < SIT; ++i) smv[i] = 1u;
                if (mask_in) {
#pragma unroll
                    for (int i = 0; i < SIT; ++i) smv[i] = mask_at(mask_in, spix_[i], packed_masks);
                    loaded_together(smv);
                }
#pragma unroll
                for (int i = 0; i < SIT; ++i)
                    if (sin_[i] && smv[i]) atomicOr(&slot_bits[ssl_[i]], 1u << skh_[i]);
            }
        }
        // set-up B: one thread per (row, tap) decides "inside the image and relevant" (for a
        // masked layer it fetches the mask byte under the tap; all of a thread's bytes are in
        // flight together)
        // (any kernel size: a loop over as many pairs as there are, kept rolled - unrolled it took the registers
        // of the whole kernel)
        const int pair_it = TAPC == 32 ? (TM * taps + NT - 1) / NT : PAIR_IT;
#pragma unroll(TAPC == 32 ? 1 : PAIR_IT)
        for (int i0 = 0; i0 < ((use_halo || self_tap) ? 0 : pair_it); i0 += PAIR_CH) {
            int prow_[PAIR_CH], ptap_[PAIR_CH], ppix_[PAIR_CH];
            bool pin_[PAIR_CH];
#pragma unroll
            for (int i = 0; i < PAIR_CH; ++i) {
                const int pair = tid + (i0 + i) * NT;
                const int r = pair / taps, t = pair - r * taps;
                const bool live = pair < TM * taps;
                const int rr = live ? r : 0;
                const int kh = t / kwid, kw = t - kh * kwid;
                const int hw = row_hw[rr];
                const int ih = (int)(int16_t)(hw & 0xffff) + kh * g.dh;
                const int iw = (hw >> 16) + kw * g.dw;
                const bool inb = live && row_p[rr] >= 0 && ih >= 0 && ih < g.h && iw >= 0 && iw < g.w;
                prow_[i] = rr;
                ptap_[i] = t;
                pin_[i] = inb;
                ppix_[i] = inb ? (row_img[rr] * g.h + ih) * g.w + iw : 0;
            }
            uint32_t mv[PAIR_CH];
#pragma unroll
            for (int i = 0; i < PAIR_CH; ++i) mv[i] = 1u;
            if (mask_in) {
                // (Instances with a pixel line use a branch per form of mask: without one their loop over the taps comes out with too few registers to hold
                // a stage's fragment addresses ahead of its barrier, and the look-ups are a small part of their long reductions: 512 -> 512 on 32 x 15 x 20, 0.1 /
                // 0.3 / 0.5 kept, 32.2 / 33.8 / 42.4 -> 30.2 / 32.0 / 41.2 us, E4M3 20.3 / 21.8 / 25.6 -> 18.6 / 20.0 / 24.4.  The tiles that label their own rows lose
                // 0.2 us with it, 512 -> 512 stride 2 from 32 x 30 x 40 1.8.)
#pragma unroll
                for (int i = 0; i < PAIR_CH; ++i) {
                    if constexpr (HALO)
                        mv[i] = packed_masks ? (reinterpret_cast<const uint32_t *>(mask_in)[ppix_[i] >> 5] >> (uint32_t)(ppix_[i] & 31)) & 1u
                                             : (uint32_t)mask_in[ppix_[i]];
                    else
                        mv[i] = mask_at(mask_in, ppix_[i], packed_masks);
                }
                if constexpr (!HALO) loaded_together(mv);
            }
#pragma unroll
            for (int i = 0; i < PAIR_CH; ++i)
                if (pin_[i] && mv[i]) atomicOr(&row_bits[prow_[i]], 1u << ptap_[i]);
        }
        // (a dropped row is marked after the bytes of all taps were requested: one round trip for both)
        if (OWN && dropped_row) row_p[tid] = -2 - sa_p;

        // per-thread, loop-invariant byte offsets; gp = the global 16-byte piece this lane
        // fetches for its LDS slot (the swizzle)
        uint32_t woff[WR];
        int wgp[WR];
#pragma unroll
        for (int j = 0; j < WR; ++j) {
            const int r = prow + j * RPP;
            const int co = co0 + r;
            wgp[j] = slot ^ FC_SWZ(r);
            woff[j] = co < g.c_out ? ((uint32_t)co * (uint32_t)(taps * g.c_in) + (PACK ? 0u : (uint32_t)wgp[j] * EPP)) * ES
                                   : kOutOfRange;
        }

        f32x16_t acc[PB][CB];
#pragma unroll
        for (int a = 0; a < PB; ++a)
#pragma unroll
            for (int b = 0; b < CB; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    acc[a][b][q * 4 + 0] = bias_q[b][q].x;
                    acc[a][b][q * 4 + 1] = bias_q[b][q].y;
                    acc[a][b][q * 4 + 2] = bias_q[b][q].z;
                    acc[a][b][q * 4 + 3] = bias_q[b][q].w;
                }

        if (HALO && use_halo) {
            // ---------------- shared-halo loop ----------------
            // LDS: two buffers of SL pixel slots, then NBW buffers of TN weight rows.  A group =
            // one (kernel row, 64-channel chunk): its pixel line is gathered once (XL wave loads
            // per thread, issued a whole group ahead), its three taps are three stages, each
            // with its own weight slab (WR wave loads per thread, issued NBW - 1 stages ahead).
            __syncthreads(); // slot_bits complete
            constexpr int XL = HALO ? SL / RPP : 1;
            constexpr uint32_t XB = (uint32_t)SL * 128u;
            constexpr uint32_t WB = (uint32_t)TN * 128u;
            // A slot's offset is that of its first kernel row, which may lie above or left of the
            // image; the load instruction adds the kernel row's offset itself and range-checks
            // the per-lane part alone, so that part must not be negative: the line is gathered
            // through a descriptor that starts (pad_h rows + pad_w pixels) before the tensor.
            // (Nothing in front of the tensor is ever read: those taps are switched off.)
            const uint32_t xbias = (uint32_t)(g.ph * g.w + g.pw) * (uint32_t)g.c_in * (uint32_t)ES;
            const u32x4_t rsrc_xb = make_rsrc_words(reinterpret_cast<const unsigned char *>(x) - xbias,
                                                    (uint32_t)g.n * g.h * g.w * g.c_in * (uint32_t)ES + xbias);
            uint32_t hxoff[XL], hxbits[XL];
            int hxgp[XL];
#pragma unroll
            for (int j = 0; j < XL; ++j) {
                const int sl = prow + j * RPP;
                hxgp[j] = slot ^ FC_SWZ(sl);
                hxoff[j] = ((uint32_t)slot_pix[sl] * (uint32_t)g.c_in + (uint32_t)hxgp[j] * EPP) * ES + xbias;
                hxbits[j] = slot_bits[sl];
            }
            // fragment addressing: the three slots of this lane's rows
            uint32_t xfa[PB][3];
#pragma unroll
            for (int a = 0; a < PB; ++a) {
                const int cs = row_cs[wave_m * WTM + a * 32 + (lane & 31)];
#pragma unroll
                for (int t = 0; t < 3; ++t) {
                    const int sl = cs + t - 1;
                    xfa[a][t] = (uint32_t)sl * 128u + (uint32_t)(((lane >> 5) * HALF) ^ FC_SWZ(sl)) * 16u;
                }
            }
            const int groups = g.kh * cchunks;
            int g_begin = 0, g_end = groups;
            if (S > 1) {
                g_begin = (int)((uint32_t)(split * groups) / (uint32_t)S);
                g_end = (int)((uint32_t)((split + 1) * groups) / (uint32_t)S);
            }
            const int ng = g_end - g_begin;
            // cursors: next pixel line to gather, next weight slab to fetch
            int xkh = g_begin / cchunks, xcc = g_begin - xkh * cchunks, xleft = ng;
            int wkh = xkh, wcc = xcc, wkw = 0, wleft = 3 * ng;
            uint32_t ld_off[WR + XL];
            // (buffer numbers are compile-time values throughout: the group loop is unrolled over
            // the two line buffers, so fragment and gather addresses inside LDS need no arithmetic)
            // Offsets of a stage's loads: a per-lane part (ld_off) and a wave-uniform part that the
            // load instruction adds itself (ld_sx for the line, ld_sw for the slab).  When the
            // input channels are whole 64-channel chunks the per-lane part of a weight row never
            // changes and that of a slot only depends on its tap-valid bit; with a channel tail
            // the lanes past the last channel are switched off one by one.
            const bool k_tail = (g.c_in % TK) != 0;
            uint32_t ld_sx = 0, ld_sw = 0;
#define FC_HALO_PREP_X(at)                                                                                \
    {                                                                                                     \
        const uint32_t sx = (uint32_t)((xkh * g.dh) * g.w * g.c_in + xcc * TK) * ES;                      \
        const bool in_k = xleft > 0;                                                                      \
        --xleft;                                                                                          \
        if (k_tail) {                                                                                     \
            ld_sx = 0;                                                                                    \
            _Pragma("unroll") for (int j = 0; j < XL; ++j)                                                \
            {                                                                                             \
                const bool ok = in_k && xcc * TK + hxgp[j] * EPP < g.c_in && ((hxbits[j] >> (xkh & 31)) & 1u); \
                ld_off[(at) + j] = ok ? hxoff[j] + sx : kOutOfRange;                                      \
            }                                                                                             \
        } else {                                                                                          \
            ld_sx = in_k ? sx : 0u;                                                                       \
            const uint32_t sel = in_k ? 1u << (xkh & 31) : 0u;                                            \
            _Pragma("unroll") for (int j = 0; j < XL; ++j)                                                \
                ld_off[(at) + j] = (hxbits[j] & sel) ? hxoff[j] : kOutOfRange;                            \
        }                                                                                                 \
        const int wrap = (xcc + 1 == cchunks);                                                            \
        xcc = wrap ? 0 : xcc + 1;                                                                         \
        xkh += wrap;                                                                                      \
    }
#define FC_HALO_PREP_W()                                                                                  \
    {                                                                                                     \
        const uint32_t sw = (uint32_t)((wkh * 3 + wkw) * g.c_in + wcc * TK) * ES;                         \
        const bool in_k = wleft > 0;                                                                      \
        --wleft;                                                                                          \
        if (k_tail) {                                                                                     \
            ld_sw = 0;                                                                                    \
            _Pragma("unroll") for (int j = 0; j < WR; ++j)                                                \
            {                                                                                             \
                const bool ok = in_k && wcc * TK + wgp[j] * EPP < g.c_in;                                 \
                ld_off[j] = ok ? woff[j] + sw : kOutOfRange;                                              \
            }                                                                                             \
        } else {                                                                                          \
            ld_sw = in_k ? sw : 0u;                                                                       \
            _Pragma("unroll") for (int j = 0; j < WR; ++j) ld_off[j] = in_k ? woff[j] : kOutOfRange;      \
        }                                                                                                 \
        const int w3 = (wkw == 2);                                                                        \
        wkw = w3 ? 0 : wkw + 1;                                                                           \
        const int wc = w3 & (wcc + 1 == cchunks);                                                         \
        wcc = w3 ? (wc ? 0 : wcc + 1) : wcc;                                                              \
        wkh += wc;                                                                                        \
    }
            // wave loads j in [first, last) of a stage's issue list: the weight slab (to ring
            // position wb) first, then, where the stage has one, the pixel line (to line buffer xb)
            const uint32_t lds_wave = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)wave * 1024u);
#define FC_HALO_ISSUE(first, last, total, xb, wb)                                                         \
    _Pragma("unroll") for (int j = (first); j < (last); ++j)                                              \
        if (j < (total))                                                                                  \
            dma_load16_s(j < WR ? rsrc_w : rsrc_xb, ld_off[j], j < WR ? ld_sw : ld_sx,                    \
                         lds_wave + (j < WR ? 2u * XB + (uint32_t)(wb) * WB + (uint32_t)j * (RPP * 128)   \
                                            : (uint32_t)(xb) * XB + (uint32_t)(j - WR) * (RPP * 128)));

            // prologue, in this order: first pixel line (to buffer 0), then NBW - 1 weight slabs
            FC_HALO_PREP_X(WR)
            FC_HALO_ISSUE(WR, WR + XL, WR + XL, 0, 0)
#pragma unroll
            for (int d = 0; d < NBW - 1; ++d) {
                FC_HALO_PREP_W()
                FC_HALO_ISSUE(0, WR, WR, 0, d)
            }
            // one group: line buffer CXB is multiplied three times; the slab of tap t sits at ring
            // position (CW0 + t) % NBW
            auto group = [&](auto cxb_c, auto cw0_c) __attribute__((always_inline)) {
                constexpr int CXB = decltype(cxb_c)::value, CW0 = decltype(cw0_c)::value;
#pragma unroll
                for (int t = 0; t < 3; ++t) {
                    const int cwb = (CW0 + t) % NBW;            // (compile-time after unrolling)
                    const int iwb = (cwb + NBW - 1) % NBW;      // ring position the slab issued now goes to
                    // this stage issues the weight slab NBW - 1 stages ahead and, on the first
                    // tap, after it, the next group's pixel line
                    FC_HALO_PREP_W()
                    if (t == 0) FC_HALO_PREP_X(WR)
                    constexpr int kBehindW = (NBW - 2) * WR; // loads issued after this stage's slab ...
                    // ... on tap 0 (the line of this group was issued before that slab); on taps
                    // 1 and 2 the next group's line is in flight behind it as well
                    if (t == 0) wait_vmcnt<kBehindW>();
                    if (t == 1) wait_vmcnt<kBehindW + XL>();
                    if (t == 2) wait_vmcnt<(NBW == 3 ? WR + XL : 0)>();
                    __syncthreads();
                    const unsigned char *xs = stage0 + (uint32_t)CXB * XB;
                    const unsigned char *ws =
                        stage0 + 2u * XB + (uint32_t)cwb * WB + (wave_n * WTN) * 128 + frag_row;
                    const int nld = t == 0 ? WR + XL : WR;
                    const int lpk = t == 0 ? (WR + XL + KK - 1) / KK : (WR + KK - 1) / KK;
                    Frag<DT> wf[FB][CB], xf[FB][PB];
#pragma unroll
                    for (int b = 0; b < CB; ++b) wf[0][b].load(ws + b * 4096, frag_t16);
#pragma unroll
                    for (int a = 0; a < PB; ++a) xf[0][a].load(xs, xfa[a][t]);
#pragma unroll
                    for (int kk = 0; kk < KK; ++kk) {
                        if (FB == 2 && kk + 1 < KK) {
                            const uint32_t o = ((uint32_t)(kk + 1) * KSTEP) ^ frag_t16;
#pragma unroll
                            for (int b = 0; b < CB; ++b) wf[(kk + 1) & 1][b].load(ws + b * 4096, o);
#pragma unroll
                            for (int a = 0; a < PB; ++a)
                                xf[(kk + 1) & 1][a].load(xs, xfa[a][t] ^ ((uint32_t)(kk + 1) * KSTEP));
                        }
                        __builtin_amdgcn_sched_barrier(0);
                        FC_HALO_ISSUE(kk * lpk, (kk + 1) * lpk, nld, CXB ^ 1, iwb)
#pragma unroll
                        for (int a = 0; a < PB; ++a)
#pragma unroll
                            for (int b = 0; b < CB; ++b)
                                acc[a][b] = mfma32<DT>(wf[kk % FB][b], xf[kk % FB][a], acc[a][b]);
                        if (FB == 1 && kk + 1 < KK) {
                            __builtin_amdgcn_sched_barrier(0);
                            const uint32_t o = ((uint32_t)(kk + 1) * KSTEP) ^ frag_t16;
#pragma unroll
                            for (int b = 0; b < CB; ++b) wf[0][b].load(ws + b * 4096, o);
#pragma unroll
                            for (int a = 0; a < PB; ++a) xf[0][a].load(xs, xfa[a][t] ^ ((uint32_t)(kk + 1) * KSTEP));
                        }
                    }
                }
            };
            // groups alternate between the two line buffers; with a ring of two slabs the ring
            // position of a group's first slab alternates as well (three stages per group), with
            // a ring of three it is always position 0
            static_assert(NBW == 2 || NBW == 3, "weight ring of the shared-halo loop");
            for (int gi = 0; gi < ng; gi += 2) {
                group(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
                if (gi + 1 < ng) group(std::integral_constant<int, 1>{}, std::integral_constant<int, (NBW == 2 ? 1 : 0)>{});
            }
#undef FC_HALO_ISSUE
#undef FC_HALO_PREP_W
#undef FC_HALO_PREP_X
        } else {
        __syncthreads(); // row_bits complete
        uint32_t xoff[XR], xbits[XR];
        int xgp[XR];
#pragma unroll
        for (int j = 0; j < XR; ++j) {
            const int r = prow + j * RPP;
            xgp[j] = slot ^ FC_SWZ(r);
            xoff[j] = ((uint32_t)row_base[r] * (uint32_t)g.c_in + (PACK ? 0u : (uint32_t)xgp[j] * EPP)) * ES;
            xbits[j] = OWN && row_p[r] < 0 ? 0u : row_bits[r];
        }
        if constexpr (OWN) {
            static_assert(TM == 64, "one lane per row");
            if (__ballot(row_p[lane] >= 0) == 0) nst = 0; // 64 rows, all irrelevant or past the end
        }
        // cursor: the next stage to be issued (starts at this unit's first stage)
        int tap = s_begin / cchunks, cc = s_begin - tap * cchunks;
        int kh = tap / kwid, kw = tap - kh * kwid;
        int to_issue = nst; // stages of this unit not yet issued
        int ibuf = 0;       // LDS buffer the next stage goes to
        // PACK: the piece of the reduction that this lane fetches (the same column of every row), its tap and its place in the tap; a
        // stage further on they are eight pieces on
        static_assert(!PACK || RPP % 16 == 0, "one swizzle for all of a lane's rows");
        int piece = 0, ptap = 0, pch = 0, step_taps = 0, step_rest = 0, kw_inv = 0;
        if constexpr (PACK) {
            piece = s_begin * 8 + (slot ^ FC_SWZ(prow));
            ptap = piece / tap_pieces;
            pch = piece - ptap * tap_pieces;
            step_taps = 8 / tap_pieces;
            step_rest = 8 - step_taps * tap_pieces;
            kw_inv = 65536 / kwid + 1; // tap / kwid, exact for the taps there are
        }

        // Offsets and LDS targets of the cursor's stage (L wave loads), then advance the cursor.
        uint32_t ld_off[L], ld_lds[L];
#define FC_PREPARE_STAGE()                                                                                \
    {                                                                                                     \
        const uint32_t sx = (uint32_t)(((kh * g.dh) * g.w + kw * g.dw) * g.c_in + cc * TK) * ES;          \
        const uint32_t sw = (uint32_t)(tap * g.c_in + cc * TK) * ES;                                      \
        const uint32_t ldsx = lds0 + (uint32_t)ibuf * STAGE_BYTES + (uint32_t)wave * 1024u;               \
        const bool in_k = to_issue > 0;                                                                   \
        --to_issue;                                                                                       \
        _Pragma("unroll") for (int j = 0; j < XR; ++j)                                                    \
        {                                                                                                 \
            const bool ok = in_k && cc * TK + xgp[j] * EPP < g.c_in && ((xbits[j] >> (tap & 31)) & 1u);   \
            ld_off[j] = ok ? xoff[j] + sx : kOutOfRange;                                                  \
            ld_lds[j] = ldsx + (uint32_t)j * (RPP * 128);                                                 \
        }                                                                                                 \
        _Pragma("unroll") for (int j = 0; j < WR; ++j)                                                    \
        {                                                                                                 \
            const bool ok = in_k && cc * TK + wgp[j] * EPP < g.c_in;                                      \
            ld_off[XR + j] = ok ? woff[j] + sw : kOutOfRange;                                             \
            ld_lds[XR + j] = ldsx + (uint32_t)(TM * 128 + j * (RPP * 128));                               \
        }                                                                                                 \
        const int wrap_c = (cc + 1 == cchunks);                                                           \
        cc = wrap_c ? 0 : cc + 1;                                                                         \
        tap += wrap_c;                                                                                    \
        const int wrap_w = wrap_c & (kw + 1 == kwid);                                                     \
        kw = wrap_c ? (wrap_w ? 0 : kw + 1) : kw;                                                         \
        kh += wrap_w;                                                                                     \
        ibuf = (ibuf + 1 == NB) ? 0 : ibuf + 1;                                                           \
    }
        // the same, pieces packed: the offsets of a row's tap and of the piece in it are the lane's own
        auto prepare_packed = [&]() __attribute__((always_inline)) {
            const int pkh = (ptap * kw_inv) >> 16, pkw = ptap - pkh * kwid;
            const uint32_t sx = (uint32_t)((pkh * g.dh * g.w + pkw * g.dw) * tap_pieces + pch) * 16u;
            const uint32_t ldsx = lds0 + (uint32_t)ibuf * STAGE_BYTES + (uint32_t)wave * 1024u;
            const bool in_k = to_issue > 0 && ptap < taps;
            --to_issue;
            const uint32_t bit = in_k ? 1u << (ptap & 31) : 0u;
#pragma unroll
            for (int j = 0; j < XR; ++j) {
                ld_off[j] = (xbits[j] & bit) ? xoff[j] + sx : kOutOfRange;
                ld_lds[j] = ldsx + (uint32_t)j * (RPP * 128);
            }
#pragma unroll
            for (int j = 0; j < WR; ++j) {
                ld_off[XR + j] = in_k ? woff[j] + (uint32_t)piece * 16u : kOutOfRange;
                ld_lds[XR + j] = ldsx + (uint32_t)(TM * 128 + j * (RPP * 128));
            }
            piece += 8;
            pch += step_rest;
            const int over = pch >= tap_pieces;
            ptap += step_taps + over;
            pch -= over ? tap_pieces : 0;
            ibuf = (ibuf + 1 == NB) ? 0 : ibuf + 1;
        };
#define FC_ISSUE_LOADS(first, last)                                                                       \
    _Pragma("unroll") for (int j = (first); j < (last); ++j)                                              \
        if (j < L) dma_load16(j < XR ? rsrc_x : rsrc_w, ld_off[j], __builtin_amdgcn_readfirstlane(ld_lds[j]));

        // prologue: NB-1 stages in flight (stages past the end are all out of range: free)
#pragma unroll
        for (int d = 0; d < NB - 1; ++d) {
            if constexpr (PACK) prepare_packed();
            else FC_PREPARE_STAGE()
            FC_ISSUE_LOADS(0, L)
        }

        constexpr int LPK = (L + KK - 1) / KK; // wave loads issued per 16-wide k-step
        int cbuf = 0;                          // buffer of the stage being multiplied
        for (int s = 0; s < nst; ++s) {
            // stage s + NB - 1: addresses only
            if constexpr (PACK) prepare_packed();
            else FC_PREPARE_STAGE()
            wait_vmcnt<(NB - 2) * L>(); // this thread's loads of stage s have landed
            __syncthreads();            // ... and everyone else's; buffer (s-1) % NB is free
            const unsigned char *xs = stage0 + cbuf * STAGE_BYTES + (wave_m * WTM) * 128 + frag_row;
            const unsigned char *ws = stage0 + cbuf * STAGE_BYTES + (TM + wave_n * WTN) * 128 + frag_row;
            Frag<DT> wf[FB][CB], xf[FB][PB];
#pragma unroll
            for (int b = 0; b < CB; ++b) wf[0][b].load(ws + b * 4096, frag_t16);
#pragma unroll
            for (int a = 0; a < PB; ++a) xf[0][a].load(xs + a * 4096, frag_t16);
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                if (FB == 2 && kk + 1 < KK) {
                    const uint32_t o = ((uint32_t)(kk + 1) * KSTEP) ^ frag_t16;
#pragma unroll
                    for (int b = 0; b < CB; ++b) wf[(kk + 1) & 1][b].load(ws + b * 4096, o);
#pragma unroll
                    for (int a = 0; a < PB; ++a) xf[(kk + 1) & 1][a].load(xs + a * 4096, o);
                }
                // keep the order "fetch step kk+1, then multiply step kk": the LDS latency
                // then hides under the MFMAs
                __builtin_amdgcn_sched_barrier(0);
                // the gathers of stage s + NB - 1 are spread over the k-steps, so that the
                // wave never queues behind a burst of loads with its matrix pipe idle
                FC_ISSUE_LOADS(kk * LPK, (kk + 1) * LPK)
#pragma unroll
                for (int a = 0; a < PB; ++a)
#pragma unroll
                    for (int b = 0; b < CB; ++b) acc[a][b] = mfma32<DT>(wf[kk % FB][b], xf[kk % FB][a], acc[a][b]);
                if (FB == 1 && kk + 1 < KK) {
                    __builtin_amdgcn_sched_barrier(0);
                    const uint32_t o = ((uint32_t)(kk + 1) * KSTEP) ^ frag_t16;
#pragma unroll
                    for (int b = 0; b < CB; ++b) wf[0][b].load(ws + b * 4096, o);
#pragma unroll
                    for (int a = 0; a < PB; ++a) xf[0][a].load(xs + a * 4096, o);
                }
            }
            cbuf = (cbuf + 1 == NB) ? 0 : cbuf + 1;
        }
#undef FC_ISSUE_LOADS
#undef FC_PREPARE_STAGE
        } // tap-by-tap loop

        // ---- epilogue: one rounding, ReLU; the tile is transposed through LDS so that every
        // lane stores 16 contiguous bytes.  First let every LDS write in flight land. ----
        wait_vmcnt<0>();
        __syncthreads();
        if (S > 1) {
            // Park this unit's fp32 partial tile (accumulator order, coalesced), then count
            // in; the unit that arrives last adds the S partials in split order - a fixed
            // order, so the result does not depend on which unit that is - and finishes the
            // tile.  Nobody waits for anybody.  The partials and the counter are written and
            // read with device-scope accesses, which go through to the memory side of the
            // per-XCD L2s, so no cache-wide write-back or invalidate is needed.
            // (16 bytes per access with the device-scope cache policy, the form a relaxed
            // agent-scope atomic store / load of 8 bytes compiles to, at twice the width)
            const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(
                partials, 0, (uint32_t)((size_t)kSplitGrid * kSplitTileFloats * sizeof(float)), 0x00020000);
            const uint32_t mine = (uint32_t)unit * (uint32_t)(TM * TN * 4);
#pragma unroll
            for (int a = 0; a < PB; ++a)
#pragma unroll
                for (int b = 0; b < CB; ++b)
#pragma unroll
                    for (int h = 0; h < 4; ++h) {
                        u32x4_t v;
                        v.x = __float_as_uint(acc[a][b][4 * h]);
                        v.y = __float_as_uint(acc[a][b][4 * h + 1]);
                        v.z = __float_as_uint(acc[a][b][4 * h + 2]);
                        v.w = __float_as_uint(acc[a][b][4 * h + 3]);
                        __builtin_amdgcn_raw_buffer_store_b128(
                            v, rp, mine + (uint32_t)(((a * CB + b) * 4 + h) * NT + tid) * 16u, 0, kDeviceScope);
                    }
            wait_vmcnt<0>(); // this thread's partial stores have been acknowledged
            __syncthreads(); // ... and every other thread's
            if (tid == 0)
                row_bits[0] = (uint32_t)__hip_atomic_fetch_add(&tile_counters[tile], 1, __ATOMIC_RELAXED,
                                                               __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            const bool last = (int)row_bits[0] == S - 1;
            if (!last) continue; // uniform: the whole workgroup moves on
            if (tid == 0)        // leave the counters as they were found
                __hip_atomic_store(&tile_counters[tile], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int a = 0; a < PB; ++a)
#pragma unroll
                for (int b = 0; b < CB; ++b)
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;
            // (several partial tiles in flight: one round trip each was most of a split tile's time)
            constexpr int U = PB * CB <= 1 ? 4 : (PB * CB <= 2 ? 2 : 1);
            for (int sp = 0; sp < S; sp += U) {
                u32x4_t v[U][PB][CB][4];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint32_t theirs = sp + u < S ? (uint32_t)(tile * S + sp + u) * (uint32_t)(TM * TN * 4) : kOutOfRange;
#pragma unroll
                    for (int a = 0; a < PB; ++a)
#pragma unroll
                        for (int b = 0; b < CB; ++b)
#pragma unroll
                            for (int h = 0; h < 4; ++h)
                                v[u][a][b][h] = __builtin_amdgcn_raw_buffer_load_b128(
                                    rp, theirs + (uint32_t)(((a * CB + b) * 4 + h) * NT + tid) * 16u, 0, kDeviceScope);
                }
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int a = 0; a < PB; ++a)
#pragma unroll
                        for (int b = 0; b < CB; ++b)
#pragma unroll
                            for (int h = 0; h < 4; ++h) {
                                acc[a][b][4 * h] += __uint_as_float(v[u][a][b][h].x);
                                acc[a][b][4 * h + 1] += __uint_as_float(v[u][a][b][h].y);
                                acc[a][b][4 * h + 2] += __uint_as_float(v[u][a][b][h].z);
                                acc[a][b][4 * h + 3] += __uint_as_float(v[u][a][b][h].w);
                            }
            }
        }
        constexpr int OP = TN * (int)sizeof(TO) + 16;
        static_assert((size_t)TM * OP <= REGION, "output tile fits");
        unsigned char *Os = smem_raw;
#pragma unroll
        for (int a = 0; a < PB; ++a) {
            const int r = wave_m * WTM + a * 32 + (lane & 31);
#pragma unroll
            for (int b = 0; b < CB; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int cl = wave_n * WTN + b * 32 + q * 8 + (lane >> 5) * 4;
                    float v0 = acc[a][b][q * 4 + 0], v1 = acc[a][b][q * 4 + 1];
                    float v2 = acc[a][b][q * 4 + 2], v3 = acc[a][b][q * 4 + 3];
                    if constexpr (sizeof(TO) == 4) {
                        if (g.flags & FC_RELU) {
                            v0 = relu_keep_nan(v0); v1 = relu_keep_nan(v1);
                            v2 = relu_keep_nan(v2); v3 = relu_keep_nan(v3);
                        }
                        store4<ODT, TO>(reinterpret_cast<TO *>(Os + r * OP) + cl, v0, v1, v2, v3);
                    } else if constexpr (sizeof(TO) == 1) {
                        // 8-bit outputs: four codes per word, the same sign-bit rule
                        uint32_t pk;
                        store4<ODT, TO>(reinterpret_cast<TO *>(&pk), v0, v1, v2, v3);
                        if (g.flags & FC_RELU) pk = relu_packed8(pk);
                        *reinterpret_cast<uint32_t *>(Os + r * OP + cl) = pk;
                    } else {
                        // 16-bit outputs: round first, then clear the values whose sign bit is set, two
                        // at a time (rounding keeps the sign, so this is max(., 0) of the rounded value)
                        uint2 pk;
                        store4<ODT, TO>(reinterpret_cast<TO *>(&pk), v0, v1, v2, v3);
                        if (g.flags & FC_RELU) {
                            pk.x = relu_packed16(pk.x);
                            pk.y = relu_packed16(pk.y);
                        }
                        *reinterpret_cast<uint2 *>(Os + r * OP + cl * 2) = pk;
                    }
                }
        }
        __syncthreads();
        constexpr int PPR = TN * (int)sizeof(TO) / 16;
        constexpr int EPT = 16 / (int)sizeof(TO);
        // a thread keeps its 16-byte column and walks down the rows; all LDS reads of the walk
        // are issued before the first store
        constexpr int RPI = NT / PPR;   // rows per pass of the workgroup
        constexpr int NPASS = TM / RPI;
        static_assert(NT % PPR == 0 && TM % RPI == 0, "store walk");
        {
            const int pc = tid % PPR, r0 = tid / PPR;
            const int co = co0 + pc * EPT;
            int pp[NPASS];
            u32x4_t pv[NPASS];
#pragma unroll
            for (int k = 0; k < NPASS; ++k) {
                const int r = r0 + k * RPI;
                pp[k] = row_p[r];
                pv[k] = *reinterpret_cast<const u32x4_t *>(Os + r * OP + pc * 16);
            }
            // streaming stores: the output is not read again by this kernel
#pragma unroll
            for (int k = 0; k < NPASS; ++k) {
                if (OWN && pp[k] < -1 && !(g.flags & FC_SKIP_ZERO_FILL)) {
                    pp[k] = -2 - pp[k];
                    pv[k] = u32x4_t{0u, 0u, 0u, 0u};
                }
                if (pp[k] >= 0 && co < g.c_out) {
                    // compacted output: row = place in the list, else the position itself
                    int64_t orow = (int64_t)pp[k];
                    if constexpr (CMP) {
                        if (g.flags & FC_COMPACT_OUT) orow = (int64_t)mt * TM + r0 + k * RPI;
                    }
                    __builtin_nontemporal_store(pv[k], reinterpret_cast<u32x4_t *>(out + orow * g.c_out + co));
                }
            }
        }
    }
