// Launches that leave most of the GPU idle, d = 64 (gfx950): two waves share 32 owner rows.
//
// Such a launch is bound by the instructions of one wave: alone on its SIMD it takes 1650 clocks for a 64-row streamed tile of
// the forward pass, four times what its contractions need.  So where there are fewer waves than SIMDs, the rows of a wave
// are given to two: each takes one of the two 32-row blocks of every streamed tile (scores, sigmoid), hands the result to
// the other through LDS, and contracts both blocks into its own half of the head dimension.  Each has half the
// instructions, no sum changes its order, and the results are the bits of the other kernels.  A workgroup is two pairs, 64
// owner rows.  Measured: 1080 clocks a tile; forward of one sequence of 1000 rows and 12 heads 15.2 -> 11.3 us, of 4096 rows and
// 2 heads 47.8 -> 33.1, its backward 70.4 -> 47.9.  What is left of a step is its barrier, the exchange and the start of its
// operands, about half of it: operands requested 3, 4 or 6 ahead, the vector work begun 1, 2 or 4 slots before the first
// contraction, the first half of a block handed over early or late are all within 1 %; tiles stored in the middle of a
// step instead of its beginning 6 % slower.
//
// One step per streamed tile t, closed by a barrier: the scores of tile t + 1, the sigmoid of tile t, the output contractions
// of tile t - 1.  Tiles are requested two to four steps before they go to LDS: a step is shorter than the way to memory.
#pragma once
#include "sigattn_kernels.hpp"

namespace sigattn {
namespace pair {

constexpr int D = 64, NW = 4, THREADS = NW * 64, BM = 64, BN = 64, LD = 72;
// LDS slots of the two streamed tensors: a tile that is only read row-wise, for scores, is read in the step behind its
// store (two slots); one that is contracted over its rows two steps later (four).  So two workgroups of FWD or DQ fit a CU.
constexpr int NBUF = 4;
constexpr long long MAX_ROW_BYTES = 2ll << 20;                         // of a row of all heads (the host takes H d up to 2^20)
constexpr int slots1(int mode) { return mode == FWD ? 2 : NBUF; }      // K (FWD, DQ), Q (DKDV)
constexpr int slots2(int mode) { return mode == DQ ? 2 : NBUF; }       // V, dO (DKDV)
constexpr size_t stream_bytes(int mode) { return (size_t)(slots1(mode) + slots2(mode)) * BN * LD * sizeof(bf16_t); }
constexpr int exchanged(int mode) { return mode == DKDV ? 2 : 1; }     // P (FWD), dS (DQ), both (DKDV)
constexpr int XCH = 4096;                                              // bytes of a tile's two blocks, one tensor, one pair
constexpr size_t lds_bytes(int mode) { return stream_bytes(mode) + (size_t)exchanged(mode) * 2 * (NW / 2) * XCH; }

// STAGES: streamed tiles on their way from memory, as the registers allow
constexpr int stages(int mode) { return mode == FWD ? 4 : 2; }

template <int MODE>
__device__ __forceinline__ void run_pass(const Params &p, const Work work, unsigned char *const smem) {
    constexpr bool HAS2 = MODE != FWD;
    constexpr int NT = HAS2 ? 2 : 1, NO = MODE == DKDV ? 2 : 1, NX = exchanged(MODE);
    constexpr int STAGES = stages(MODE), S1 = slots1(MODE), S2 = slots2(MODE);
    constexpr int Y2 = S1 * BN * LD;                                   // elements from the first streamed tensor to the second
    constexpr int NA = 4 * NT, NC = 4 * NO, M = NA + NC;
    constexpr float LOG2E = 1.4426950408889634f;
    const int z = __builtin_amdgcn_readfirstlane(work.z), n = __builtin_amdgcn_readfirstlane(work.n);
    const int h = __builtin_amdgcn_readfirstlane(work.h), m0 = __builtin_amdgcn_readfirstlane(work.m0);
    const size_t row_stride = (size_t)p.H * D;
    const size_t base_o = (size_t)z * p.N * row_stride + (size_t)h * D, base_s = (size_t)z * p.N_str * row_stride + (size_t)h * D;
    int ns = n;
    if (p.seqlens_str != p.seqlens || p.N_str != p.N) {
        ns = p.seqlens_str[z];
        ns = ns < 0 ? 0 : (ns > p.N_str ? p.N_str : ns);
    }
    ns = __builtin_amdgcn_readfirstlane(ns);
    if (m0 >= n || ns == 0) {                                          // padding, or nothing to stream: zeros
        const int m1 = m0 + BM < p.N ? m0 + BM : p.N;
        zero_rows<D, THREADS>(p.out0, base_o, row_stride, m0, m1);
        if (MODE == DKDV) zero_rows<D, THREADS>(p.out1, base_o, row_stride, m0, m1);
        return;
    }
    const bf16_t *const x1 = MODE == DKDV ? p.k : p.q, *const x2 = MODE == DKDV ? p.v : p.d_o;
    const bf16_t *const y1 = MODE == DKDV ? p.q : p.k, *const y2 = MODE == DKDV ? p.d_o : p.v;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int pr = wave >> 1, half = wave & 1;                         // which pair; which block of a tile, which half of the head dimension
    const int c = lane & 31, g = lane >> 5;
    const float c1 = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, -p.scale * LOG2E)));
    const float cb = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int,
        __builtin_amdgcn_exp2f(__builtin_fminf(__builtin_fmaxf(-p.bias[z] * LOG2E, -126.0f), 126.0f)))));

    // ---- owner rows (B operands): row c of the pair's 32, columns 16 ks + 8 g + 0..7; zeros behind the last valid row
    const int row_off = (int)(((unsigned)(pr * 32 + c) * (unsigned)row_stride + 8u * g) * 2u);
    bf16x8 xa[4], xb[HAS2 ? 4 : 1];
    {
        const int rows = n - m0 < BM ? n - m0 : BM;
        const int bytes = __builtin_amdgcn_readfirstlane(rows * (int)row_stride * 2);
        const auto d1 = __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(x1 + base_o + (size_t)m0 * row_stride), 0, bytes, 0x00027000);
        const auto d2 = __builtin_amdgcn_make_buffer_rsrc(uniform_ptr((HAS2 ? x2 : x1) + base_o + (size_t)m0 * row_stride), 0, bytes, 0x00027000);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            xa[ks] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(d1, row_off + 32 * ks, 0, 0));
            if (HAS2) xb[HAS2 ? ks : 0] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(d2, row_off + 32 * ks, 0, 0));
        }
    }

    // ---- streamed tiles: HBM -> registers -> LDS; a thread moves rows r0 and r0 + 32
    bf16_t *const y1s = reinterpret_cast<bf16_t *>(smem);
    const int ntiles = (ns + BN - 1) / BN;
    const int r0 = tid >> 3, col0 = (tid & 7) * 8;
    const int ld_off = (int)(((unsigned)r0 * (unsigned)row_stride + (unsigned)col0) * 2u);
    const unsigned pass = 32u * (unsigned)row_stride * 2u;
    // one descriptor per tensor, ending with the last valid row: what lies behind it reads as zeros (the host keeps a head's
    // rows below 2^31 bytes)
    const int str_bytes = __builtin_amdgcn_readfirstlane(ns * (int)row_stride * 2);
    const auto ds1 = __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(y1 + base_s), 0, str_bytes, 0x00027000);
    const auto ds2 = __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(y2 + base_s), 0, str_bytes, 0x00027000);
    // Bytes to the tile that is requested next.  Tiles are requested up to STAGES + 2 behind the last one (they read as zeros), so
    // this may pass 2^31; with its lane's offset it stays below 2^32.
    unsigned at = 0;
    static_assert((1ll << 31) + (STAGES + 4) * BN * MAX_ROW_BYTES < 1ll << 32, "offsets of requested tiles in 32 bits");
    u32x4 st[STAGES][4];
    auto load_tile = [&](auto stage_c) {
        constexpr int S = decltype(stage_c)::value % STAGES;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            st[S][i] = __builtin_amdgcn_raw_buffer_load_b128(ds1, ld_off, (int)(at + i * pass), 0);
            st[S][2 + i] = __builtin_amdgcn_raw_buffer_load_b128(ds2, ld_off, (int)(at + i * pass), 0);
        }
        at += 2 * pass;
    };
    bf16_t *const w = y1s + r0 * LD + col0;
    auto store_tile = [&](auto slot_c) {                               // slot: the tile's number modulo NBUF, which its stage and places follow from
        constexpr int slot = decltype(slot_c)::value, S = slot % STAGES;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            *reinterpret_cast<u32x4 *>(w + (slot % S1 * BN + 32 * i) * LD) = st[S][i];
            *reinterpret_cast<u32x4 *>(w + (slot % S2 * BN + 32 * i) * LD + Y2) = st[S][2 + i];
        }
    };
    static_assert(NBUF % STAGES == 0, "a slot has one stage");

    // ---- LDS addresses: this wave's block row-wise, its columns transposed, the exchange of its pair
    const int i16 = lane & 15, g16 = (lane >> 4) & 1;
    const bf16_t *const rd = y1s + (32 * half + c) * LD + 8 * g;
    const bf16_t *const tr = y1s + (4 * g + (i16 >> 2)) * LD + 32 * half + 16 * g16 + 4 * (i16 & 3);
    unsigned char *const xch = smem + stream_bytes(MODE) + pr * XCH + lane * 16;     // [tensor][parity][pair][block][half of the block][lane]
    unsigned char *const xch_mine = xch + half * 2048;
    constexpr int XPAR = (NW / 2) * XCH, XTEN = 2 * XPAR;

    f32x16 acc[NO], sbuf[2], dbuf[2];
    u32x4 pw[2], dsw[2];                                               // P and dS of the block in hand, packed
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    constexpr int OPU = MODE == FWD ? 7 : (MODE == DQ ? 13 : 14), UNITS = 8;
    constexpr int AHEAD = 3;                                           // operands on their way from LDS
    constexpr int LEAD = 2;                                            // slots of vector work before the first contraction
    const int tail = ns - (ntiles - 1) * BN - 32 * half;               // valid rows of this wave's block of the last tile
    auto barrier = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    auto give = [&](auto i_, auto slot_c) {                            // half i of this block's P and dS to both waves of the pair
        constexpr int i = decltype(i_)::value, PAR = decltype(slot_c)::value & 1;
        // tensor 0 meets the first output (O, dQ, dK), tensor 1 the second (dV)
        *reinterpret_cast<u32x4 *>(xch_mine + PAR * XPAR + 1024 * i) = MODE == FWD ? pw[i] : dsw[i];
        if (NX == 2) *reinterpret_cast<u32x4 *>(xch_mine + XTEN + PAR * XPAR + 1024 * i) = pw[i];
    };
    // One step on the tile of ring slot `slot`.
    auto step = [&](auto has_prev_c, auto has_next_c, auto drain_c, auto slot_c, auto moves_c) {
        constexpr bool HAS_PREV = decltype(has_prev_c)::value, HAS_NEXT = decltype(has_next_c)::value, DRAIN = decltype(drain_c)::value;
        constexpr int slot = decltype(slot_c)::value, PAR = slot & 1;
        constexpr int LO = HAS_NEXT ? 0 : NA, HI = HAS_PREV ? M : NA;  // contractions [LO, HI) of: NA scores, NC outputs
        constexpr int SLOTS = HI - LO + LEAD;
        constexpr ValuOrder<UNITS, OPU, 2, 6> order{};
        constexpr int LEN = DRAIN ? 0 : UNITS * OPU;
        constexpr bool MOVES = decltype(moves_c)::value;               // a tile to LDS, one from memory, this block to the pair
        constexpr int GIVE_AT = [&] {                                  // the slot that packs the last pair of the block's first half
            int last = 0;
            for (int i = 0; i < UNITS * OPU; ++i)
                if (order.unit[i] == 3) last = i;
            int k = 0;
            while (((k + 1) * LEN) / SLOTS <= last && k < SLOTS - 1) ++k;
            return k;
        }();
        bf16x8 a[AHEAD], b[AHEAD];
        float pv[UNITS][2];
        auto fetch = [&](auto j_) {
            constexpr int j = decltype(j_)::value;
            if constexpr (j < NA) {                                    // scores of the next tile
                constexpr int ks = j / NT, which = j % NT, row = (slot + 1) % (which == 0 ? S1 : S2) * BN;
                a[j % AHEAD] = lds_read_rows(rd + row * LD + 16 * ks + which * Y2);
            } else {                                                   // outputs of the tile before: 16 rows each
                constexpr int q = (j - NA) / NO, which = (j - NA) % NO, row = (slot + 3) % NBUF * BN + 16 * q;
                // FWD contracts V^T (second tensor); DQ K^T (first); DKDV Q^T (first) with dS for dK, dO^T (second) with P for dV
                constexpr bool second = MODE == FWD || (MODE == DKDV && which == 1);
                const bf16_t *const t = tr + row * LD + (second ? Y2 : 0);
                a[j % AHEAD] = lds_read_tr(t, t + 8 * LD);
                b[j % AHEAD] = *reinterpret_cast<const bf16x8 *>(xch + which * XTEN + (PAR ^ 1) * XPAR + q * 1024);
            }
        };
        static_for<LO, (LO + AHEAD < HI ? LO + AHEAD : HI)>([&](auto j_) { fetch(j_); });
        static_for<0, SLOTS>([&](auto k_) {
            constexpr int k = decltype(k_)::value;
            if constexpr (k >= LEAD) {
                constexpr int j = LO + k - LEAD;
                if constexpr (j < NA) {
                    constexpr int ks = j / NT, which = j % NT;
                    if constexpr (which == 0)
                        sbuf[PAR ^ 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[j % AHEAD], xa[ks], ks == 0 ? zero : sbuf[PAR ^ 1], 0, 0, 0);
                    else
                        dbuf[PAR ^ 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[j % AHEAD], xb[HAS2 ? ks : 0], ks == 0 ? zero : dbuf[PAR ^ 1], 0, 0, 0);
                } else {
                    constexpr int which = (j - NA) % NO;
                    acc[which] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[j % AHEAD], b[j % AHEAD], acc[which], 0, 0, 0);
                }
                if constexpr (j + AHEAD < HI) fetch(IntC<j + AHEAD>{});
            }
            static_for<(k * LEN) / SLOTS, ((k + 1) * LEN) / SLOTS>([&](auto i_) {
                constexpr int i = decltype(i_)::value, u = order.unit[i], o = order.op[i], ra = 2 * u, rb = 2 * u + 1;
                f32x16 &s = sbuf[PAR];
                f32x16 &dp = dbuf[PAR];
                if constexpr (o == 0) s[ra] = __builtin_amdgcn_exp2f(s[ra]);
                else if constexpr (o == 1) s[rb] = __builtin_amdgcn_exp2f(s[rb]);
                else if constexpr (o == 2) pv[u][0] = __builtin_fmaf(cb, s[ra], 1.0f);
                else if constexpr (o == 3) pv[u][1] = __builtin_fmaf(cb, s[rb], 1.0f);
                else if constexpr (o == 4) pv[u][0] = __builtin_amdgcn_rcpf(pv[u][0]);
                else if constexpr (o == 5) pv[u][1] = __builtin_amdgcn_rcpf(pv[u][1]);
                else if constexpr (MODE == FWD) pw[u / 4][u % 4] = pack_bf16(pv[u][0], pv[u][1]);
                else if constexpr (o == 6) s[ra] = mul_zero_wins(s[ra], pv[u][0]);
                else if constexpr (o == 7) s[rb] = mul_zero_wins(s[rb], pv[u][1]);
                else if constexpr (o == 8) dp[ra] = pv[u][0] * dp[ra];
                else if constexpr (o == 9) dp[rb] = pv[u][1] * dp[rb];
                else if constexpr (o == 10) dp[ra] = s[ra] * dp[ra];
                else if constexpr (o == 11) dp[rb] = s[rb] * dp[rb];
                else if constexpr (o == 12) dsw[u / 4][u % 4] = pack_bf16(dp[ra], dp[rb]);
                else pw[u / 4][u % 4] = pack_bf16(pv[u][0], pv[u][1]);
            });
            if constexpr (MOVES && k == GIVE_AT) give(IntC<0>{}, slot_c);
            if constexpr (MOVES && k == 0) {
                store_tile(IntC<(slot + 2) % NBUF>{});
                load_tile(IntC<(slot + 2) % NBUF>{});
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (MOVES) give(IntC<1>{}, slot_c);
    };
    auto mask = [&]() {                                                // rows of the last tile behind the valid length
        if (tail >= 32) return;                                        // uniform
        const short valid = (short)(tail - 4 * g);
        const s16x2 limit = {valid, valid};
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const short row = (short)(8 * (u / 2) + 2 * (u % 2));
            const s16x2 rows = {row, (short)(row + 1)};
            const unsigned keep = __builtin_bit_cast(unsigned, (s16x2)((rows - limit) >> 15));
            if (MODE != DQ) pw[u / 4][u % 4] &= keep;
            if (HAS2) dsw[u / 4][u % 4] &= keep;
        }
    };
    using T_ = IntC<1>;
    using F_ = IntC<0>;

    // ---- prologue: tiles 0 and 1 into the ring, the next ones on their way
    static_for<0, STAGES>([&](auto t_) { load_tile(t_); });
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) xa[ks] = scale_bf16x8(xa[ks], c1);
    store_tile(IntC<0>{});
    store_tile(IntC<1>{});
    load_tile(IntC<0>{});
    load_tile(IntC<1>{});
#pragma unroll
    for (int o = 0; o < NO; ++o)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[o][i] = 0.f;
    barrier();
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        sbuf[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_read_rows(rd + 16 * ks), xa[ks], ks == 0 ? zero : sbuf[0], 0, 0, 0);
        if (HAS2) dbuf[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_read_rows(rd + 16 * ks + Y2), xb[HAS2 ? ks : 0], ks == 0 ? zero : dbuf[0], 0, 0, 0);
    }
    if constexpr (S1 == 2 || S2 == 2) barrier();                       // the first step overwrites tile 0 of a tensor with two slots
    // A step that has a tile behind it: tile t + 2 goes to its slot, last read (as the tile before) in step t - 1, and the tile STAGES
    // behind it is requested into its registers.
    auto body = [&](auto prev_c, auto slot_c) {
        step(prev_c, T_{}, F_{}, slot_c, T_{});
        barrier();
    };
    auto last = [&](auto prev_c, auto slot_c) {
        step(prev_c, F_{}, F_{}, slot_c, F_{});
        mask();
        give(IntC<0>{}, slot_c);
        give(IntC<1>{}, slot_c);
        barrier();
        step(T_{}, F_{}, T_{}, IntC<(decltype(slot_c)::value + 1) % NBUF>{}, F_{});
    };
    if (ntiles == 1) {
        last(F_{}, IntC<0>{});
    } else {
        body(F_{}, IntC<0>{});
        int t = ntiles - 2, slot = 1;                                  // steps with a tile behind them that are left
        while (t > 0) {
            if (slot == 1) { body(T_{}, IntC<1>{}); slot = 2; --t; }
            if (t > 0 && slot == 2) { body(T_{}, IntC<2>{}); slot = 3; --t; }
            if (t > 0 && slot == 3) { body(T_{}, IntC<3>{}); slot = 0; --t; }
            if (t > 0 && slot == 0) { body(T_{}, IntC<0>{}); slot = 1; --t; }
        }
        if (slot == 0) last(T_{}, IntC<0>{});
        else if (slot == 1) last(T_{}, IntC<1>{});
        else if (slot == 2) last(T_{}, IntC<2>{});
        else last(T_{}, IntC<3>{});
    }

    // ---- epilogue: columns 32 half + 16 i + 8 g + 0..7 of row c, lanes 32 apart exchange halves (as in the other kernels)
    const int rows = p.N - m0 < BM ? p.N - m0 : BM;
    const int bytes = __builtin_amdgcn_readfirstlane(rows * (int)row_stride * 2);
    const bool ok = m0 + pr * 32 + c < n;
    const float oscale = MODE == FWD ? 1.0f : p.scale * cb;
#pragma unroll
    for (int o = 0; o < NO; ++o) {
        bf16_t *const out = o == 0 ? p.out0 : p.out1;
        const auto d = __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(out + base_o + (size_t)m0 * row_stride), 0, bytes, 0x00027000);
        const float f = o == 0 ? oscale : 1.0f;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const f32x16 &v = acc[o];
            const unsigned e0 = pack_bf16(v[8 * i + 0] * f, v[8 * i + 1] * f), e1 = pack_bf16(v[8 * i + 2] * f, v[8 * i + 3] * f);
            const unsigned o0 = pack_bf16(v[8 * i + 4] * f, v[8 * i + 5] * f), o1 = pack_bf16(v[8 * i + 6] * f, v[8 * i + 7] * f);
            const auto s0 = __builtin_amdgcn_permlane32_swap(e0, o0, false, false);
            const auto s1 = __builtin_amdgcn_permlane32_swap(e1, o1, false, false);
            const u32x4 r = {s0[0], s1[0], s0[1], s1[1]}, z4 = {0u, 0u, 0u, 0u};
            __builtin_amdgcn_raw_buffer_store_b128(ok ? r : z4, d, row_off + 2 * (32 * half + 16 * i), 0, 0);
        }
    }
}

template <int MODE>
__global__ void __launch_bounds__(THREADS, 2) sigattn_pair(const Params p) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ MapScratch scratch;
    run_pass<MODE>(p, map_work<BM, THREADS>(p, blockIdx.x, scratch), smem);
}

// Both passes of the backward in one launch: workgroups [0, first_tiles) take the dK/dV tiles, or with `q_first` the dQ tiles.
__global__ void __launch_bounds__(THREADS, 2) sigattn_pair_bwd(const Params kv, const Params q, const int q_first, const int first_tiles) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ MapScratch scratch;
    const int id = blockIdx.x;
    const bool is_kv = (id < first_tiles) != (q_first != 0);
    const int rest = id < first_tiles ? id : id - first_tiles;
    if (is_kv) run_pass<DKDV>(kv, map_work<BM, THREADS>(kv, rest, scratch), smem);
    else run_pass<DQ>(q, map_work<BM, THREADS>(q, rest, scratch), smem);
}

}  // namespace pair

// d = 128, launches of at most a workgroup to a CU: forward and dQ passes of sigattn_kernel with four waves and 128 owner rows
// instead of eight and 256, so that each wave has a SIMD of its own, and the backward pass as one launch (dK/dV has 128
// owner rows there too), so that its halves run beside each other and not one after the other.  The bits are the same.
// us: forward of 8 heads of 1000 rows 26.8 -> 22.0, of 2 x 2 of 256 11.8 -> 9.4; backward 71.4 -> 33.8 and 29.4 -> 13.8 (with dQ in smaller
// workgroups but a launch of its own 61.7 and 25.2).
namespace half128 {

constexpr int NW = 4, OCC_FWD = 2, OCC_BWD = 1;      // with 256 registers the dQ pass spills 121

template <int MODE, int LD1, int LD2, int OCC>
__global__ void __launch_bounds__(NW * 64, OCC) sigattn_half(const Params p) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ MapScratch scratch;
    using C = Cfg<MODE, 128, 1, NW, 64, LD1, LD2, 4>;
    sigattn::run_pass<MODE, 128, 1, NW, 64, LD1, LD2, 4, false>(p, map_work<C::BM, C::THREADS>(p, blockIdx.x, scratch), smem, nullptr);
}

__global__ void __launch_bounds__(NW * 64, OCC_BWD) sigattn_half_bwd(const Params kv, const Params q, const int q_first, const int first_tiles) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ MapScratch scratch;
    const int id = blockIdx.x;
    const bool is_kv = (id < first_tiles) != (q_first != 0);
    const int rest = id < first_tiles ? id : id - first_tiles;
    constexpr int BM = NW * 32, THREADS = NW * 64;
    if (is_kv) sigattn::run_pass<DKDV, 128, 1, NW, 64, 144, 144, 4, false>(kv, map_work<BM, THREADS>(kv, rest, scratch), smem, nullptr);
    else sigattn::run_pass<DQ, 128, 1, NW, 64, 144, 136, 4, false>(q, map_work<BM, THREADS>(q, rest, scratch), smem, nullptr);
}

}  // namespace half128
}  // namespace sigattn
