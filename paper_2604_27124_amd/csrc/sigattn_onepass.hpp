// The backward pass of d = 64 in one pass over the scores (gfx950).
//
// The paper's two kernels (appendix Alg. 2 and Alg. 3) compute the scores, the sigmoid and dP twice: seven contractions
// and two sigmoids per pair of rows.  Here a workgroup owns 256 keys, as in Alg. 3, streams the queries and dO once and
// also forms dQ from the dS it has: five contractions and one sigmoid.  dQ of a query tile is then a sum over the
// workgroups of a head; it is passed on from one to the next in fp32, in the order of the keys, through a scratch buffer:
//
//   key tile j waits until key tile j - 1 has published tile t, starts its contraction from those sums and publishes
//   the new ones; the last one writes dQ.
//
// So the order of the sums is fixed, nothing is added atomically, and results are the same bits in every run.
//
// Every wait ends, in whatever order the hardware starts workgroups and whatever else runs on the GPU: the plan gives a
// workgroup a head, and which of its key tiles is the next that none has taken when it starts.  So the tile it waits for has been
// taken by a workgroup that has started, which keeps its CU until it ends, and the first tile waits for none.  (With the tile from
// the workgroup's id too it would not: the XCDs start workgroups each for itself, and two launches on two streams could each
// fill an XCD with workgroups that wait for one queued behind the other's.)  The tile is asked for while the first queries are on
// their way, which costs 0 to 1 % (step of 4 x 12 heads of up to 8192 rows 1360 -> 1366 us, 512 x 12 of up to 512 1034 -> 1044).  A counter for the
// whole plan, whose answer everything waits for: 512 x 12 x 512 3 % slower, 32 x 32 x 384 4 % and 16 x 12 of up to 4096 2 % faster.
//
// dS changes hands through LDS: the accumulators of a wave hold 32 keys by 32 queries with the queries along the registers,
// and dQ contracts over the keys of all eight waves.  A query tile has four 32 x 32 blocks of dQ; four waves take the
// blocks of the even tiles, the other four those of the odd ones, so that each SIMD has one wave with and one without.
//
// What bounds it: the vector pipe (2600 clocks per 64 x 256 tile and SIMD of 4900 measured), the matrix pipe (2560) and the
// LDS (2700) together, at the chip's power limit.  Backward of 4 x 12 heads of 8192 valid rows 2790 -> 2240 us, of
// 8 x 12 x 2048 368 -> 294 us (both passes in one launch before).
#pragma once
#include "sigattn_kernels.hpp"
#include "sigattn_onepass_plan.hpp"

namespace sigattn {
namespace onepass {

constexpr int D = 64;
constexpr int NW = 8, THREADS = NW * 64;     // waves of 32 keys each
static_assert(BM == NW * 32, "key rows of a workgroup");
constexpr int RING_TILES = 3;                // LDS ring: tile t lives in slot t % 3
constexpr int LD = 72;                       // elements of a streamed row in LDS
constexpr int LDT = BM + 8;                  // elements of a row of the transposed key tile
constexpr int RING = 4;                      // A operands on their way from LDS
constexpr int SLOTS = 16;                    // 32-wide MFMAs of a step (without those of dQ)
constexpr size_t STREAM_BYTES = (size_t)RING_TILES * BN * LD * 2 * sizeof(bf16_t);
constexpr size_t KT_BYTES = (size_t)D * LDT * sizeof(bf16_t);
constexpr size_t DS_BYTES = (size_t)BM * BN * sizeof(bf16_t);      // one of two
constexpr size_t LDS_BYTES = STREAM_BYTES + KT_BYTES + 2 * DS_BYTES + 1024;   // the last for dS of keys behind the end
constexpr int TILE_BYTES = BN * D * 4;       // partial sums of a query tile
constexpr int FLAGS = NW;                    // progress counters of a workgroup

struct Params {
    const bf16_t *q, *k, *v, *d_o;           // q, d_o [B, L_q, H, D];  k, v [B, L_k, H, D]
    bf16_t *dq, *dk, *dv;
    const int32_t *seqlens_q, *seqlens_k;
    const float *bias;
    float scale;
    int B, L_q, L_k, H;
    int group;                               // sequences whose tiles are dealt in turn
    TileWork *plan;                          // [B H key tiles]
    int *flags;                              // [B][H][key tiles][FLAGS]; those of a head's last tile, which no tile follows,
                                             // hold the number of its tiles that have been taken
    unsigned char *part;                     // [B][H][query tiles][TILE_BYTES]
};

// The plan of a launch (sigattn_onepass_plan.hpp): the work of every workgroup, and its progress counts set to zero.  Made by a
// kernel of its own, a thread per tile: in the workgroups themselves it took 5000 to 7000 clocks of each one's 26000 (N = 128) to
// 170000 (N = 2048).
__global__ void __launch_bounds__(PLAN_THREADS) sigattn_onepass_plan(const Params p) {
    __shared__ PlanScratch s;
    const int T = (p.L_k + BM - 1) / BM, tid = threadIdx.x;
    if (p.B <= PLAN_B) {
        const int q = tid < p.B ? p.seqlens_q[tid] : 0, k = tid < p.B ? p.seqlens_k[tid] : 0;
        plan_take(s, tid, p.B, q, p.L_q);
        __syncthreads();
        plan_rank(s, tid, p.B, k, p.L_k);
        __syncthreads();
        plan_fill(s, tid, p.B, k, p.L_k);
        for (int step = 0; step < PLAN_SCANS; ++step) {
            __syncthreads();
            plan_scan(s, tid, step);
        }
        __syncthreads();
    }
    const int i = blockIdx.x * PLAN_THREADS + tid;                   // = ((z H) + h) T + j
    if (i >= p.B * p.H * T) return;
    const int j = i % T, h = i / T % p.H, z = i / T / p.H;
    const TileWork w = {z, h, j, clamp_len(p.seqlens_q[z], p.L_q), clamp_len(p.seqlens_k[z], p.L_k), p.bias[z]};
    p.plan[plan_id(s, z, h, j, p.B, p.H, T, p.group)] = w;
    const u32x4 z4 = {0u, 0u, 0u, 0u};
    u32x4 *const counts = reinterpret_cast<u32x4 *>(p.flags + (size_t)i * FLAGS);
    counts[0] = z4;
    counts[1] = z4;
}

constexpr int SC1 = 16;              // cache policy of a buffer access: agent scope (stores write through, loads miss)
constexpr int MAX_SPINS = 1 << 24;   // of a wait, each above a microsecond: far beyond any real one, so that a fault ends as NaN in dQ, not as a hang


__global__ void __launch_bounds__(THREADS, 2) sigattn_onepass(const Params p) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr float LOG2E = 1.4426950408889634f;
    const TileWork work = p.plan[blockIdx.x];
    const int z = __builtin_amdgcn_readfirstlane(work.z), h = __builtin_amdgcn_readfirstlane(work.h);
    int j = __builtin_amdgcn_readfirstlane(work.j);
    const int nq = __builtin_amdgcn_readfirstlane(work.nq), nk = __builtin_amdgcn_readfirstlane(work.nk);
    const int T = (p.L_k + BM - 1) / BM, TQ = (p.L_q + BN - 1) / BN;
    const size_t row_stride = (size_t)p.H * D;
    const size_t base_q = (size_t)z * p.L_q * row_stride + (size_t)h * D;
    const size_t base_k = (size_t)z * p.L_k * row_stride + (size_t)h * D;
    int m0 = j * BM;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ntiles = nk > 0 ? (nq + BN - 1) / BN : 0;      // streamed tiles
    const int key_tiles = (nk + BM - 1) / BM;
    auto zero_dq_share = [&]() {                             // query rows behind the last tile, shared by the workgroups of a head
        const int from = ntiles * BN, rows = p.L_q - from;
        if (rows <= 0) return;
        const int each = (rows + T - 1) / T, a = from + j * each, b = a + each < p.L_q ? a + each : p.L_q;
        if (a < b) zero_rows<D, THREADS>(p.dq, base_q, row_stride, a, b);
    };
    if (m0 >= nk || nq == 0) {
        const int m1 = m0 + BM < p.L_k ? m0 + BM : p.L_k;
        zero_rows<D, THREADS>(p.dk, base_k, row_stride, m0, m1);
        zero_rows<D, THREADS>(p.dv, base_k, row_stride, m0, m1);
        zero_dq_share();
        return;
    }
    bf16_t *const y1s = reinterpret_cast<bf16_t *>(smem);             // Q tiles [RING_TILES][BN][LD]
    bf16_t *const y2s = y1s + RING_TILES * BN * LD;                   // dO tiles
    bf16_t *const kts = y2s + RING_TILES * BN * LD;                   // K^T [D][LDT]; behind it dS [2][BM][BN]
    const int lane = tid & 63;
    const int c = lane & 31, g = lane >> 5;
    const float c1 = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, -p.scale * LOG2E)));
    const float cb = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int,
        __builtin_amdgcn_exp2f(__builtin_fminf(__builtin_fmaxf(-work.bias * LOG2E, -126.0f), 126.0f)))));

    // ---- streamed tiles
    const int r0 = tid >> 3, col0 = (tid & 7) * 8;
    const unsigned ld_off0 = ((unsigned)r0 * (unsigned)row_stride + (unsigned)col0) * 2u;
    const bf16_t *next1 = p.q + base_q, *next2 = p.d_o + base_q;
    int rows_left = nq;
    u32x4 st1, st2;
    auto load_tile = [&]() {
        const int bytes = __builtin_amdgcn_readfirstlane((rows_left < BN ? rows_left : BN) * (int)row_stride * 2);
        const auto d1 = __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(next1), 0, bytes, 0x00027000);
        const auto d2 = __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(next2), 0, bytes, 0x00027000);
        st1 = __builtin_amdgcn_raw_buffer_load_b128(d1, (int)ld_off0, 0, 0);
        st2 = __builtin_amdgcn_raw_buffer_load_b128(d2, (int)ld_off0, 0, 0);
        next1 += (size_t)BN * row_stride;
        next2 += (size_t)BN * row_stride;
        rows_left = rows_left > BN ? rows_left - BN : 0;
    };
    bf16_t *const w1 = y1s + r0 * LD + col0;
    constexpr int Y2 = RING_TILES * BN * LD;                          // elements from the Q tiles to the dO tiles
    auto store_tile = [&](int slot) {
        *reinterpret_cast<u32x4 *>(w1 + slot * BN * LD) = st1;
        *reinterpret_cast<u32x4 *>(w1 + slot * BN * LD + Y2) = st2;
    };

    // ---- LDS addresses
    const int i16 = lane & 15, g16 = (lane >> 4) & 1;
    const bf16_t *const rd = y1s + c * LD + 8 * g;
    const bf16_t *const tr = y1s + (4 * g + (i16 >> 2)) * LD + 16 * g16 + 4 * (i16 & 3);
    // dS: element (key, q') at key * 128 + (2 q' ^ X(key)), X = 16 b2 + 32 b3 + 64 b1 of the key's bits; q' counts the 64 rows
    // of a tile so that the rows of a lane's four packed pairs are neighbours: q' = 32 nb + 16 A + 8 g + 4 (a & 1) + i for row 32 nb + 8 a + 4 g + i, A = a / 2
    const int key = wave * 32 + c;
    auto swz = [](int k) { return 16 * ((k >> 2) & 1) + 32 * ((k >> 3) & 1) + 64 * ((k >> 1) & 1); };
    const int ds_base = (int)(STREAM_BYTES + KT_BYTES);
    const int job = wave & 3, grp = wave >> 2, nbq = job & 1, dh = job >> 1;      // dQ block of this wave, and which tiles' (every second)
    const bf16_t *const kt = kts + (32 * dh + c) * LDT + 8 * g;
    const int kr = 8 * g + (i16 >> 2);                                             // + 4 for the second read
    const int dsr0 = ds_base + grp * (int)DS_BYTES + kr * 128 + ((64 * nbq + 32 * g16 + 8 * (i16 & 3)) ^ swz(kr));
    const int dsr1 = ds_base + grp * (int)DS_BYTES + (kr + 4) * 128 + ((64 * nbq + 32 * g16 + 8 * (i16 & 3)) ^ swz(kr + 4));

    bf16x8 xa[4], xb[4];                                              // owner rows: lane holds row c of its wave's 32, columns 16 ks + 8 g + 0..7
    f32x16 acc0[2], acc1[2], dqa;
    f32x16 sbuf[2], dbuf[2];
    u32x4 pbuf[2][2], dsbuf[2][2];
    bf16x8 ring[RING], qa, qb;
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

    auto barrier = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    // ---- the first queries are requested, and the tile of keys is taken
    load_tile();
    const u32x4 f1 = st1, f2 = st2;
    __builtin_amdgcn_sched_barrier(0);
    if (key_tiles > 1) {
        __shared__ int taken;
        if (tid == 0) taken = __hip_atomic_fetch_add(p.flags + (((size_t)z * p.H + h) * T + T - 1) * FLAGS, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        barrier();
        j = __builtin_amdgcn_readfirstlane(taken);
        m0 = j * BM;
    }
    const bool key_ok = m0 + key < nk;
    int dsw = key_ok ? ds_base + key * 128 + ((16 * g) ^ swz(key)) : ds_base + 2 * (int)DS_BYTES + 128 * (wave & 7) + 16 * g;
    const int flip = key_ok ? (int)DS_BYTES : 0;
    // ---- the chain of partial dQ sums
    const bool chained = j > 0, last_of_chain = j == key_tiles - 1;
    unsigned char *part = p.part + ((size_t)z * p.H + h) * TQ * (size_t)TILE_BYTES + (size_t)grp * TILE_BYTES;   // this wave's next tile
    int *const my_flag = p.flags + ((((size_t)z * p.H + h) * T + j) * FLAGS + wave);
    int avail = 0;                                                    // tiles the workgroup of the keys before has published
    bool lost = false;                                                // a wait was given up
    const int part_off = job * 4096 + lane * 16;
    // Published tiles are counted by each wave for itself: the wave of the next workgroup that adds to a block is the one of the
    // same number, with the same lanes at the same places.  The sums are written through and read past the caches (the workgroups
    // of a head may run on different XCDs); a count follows when the stores it stands for are done.  The count is looked at most
    // of a tile before the sums are wanted and only waited for where that look came too early.
    auto look = [&]() { return __hip_atomic_load(my_flag - FLAGS, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    int seen = 0;                                                     // what the last look found, not waited for
    auto dq_look = [&]() { if (chained) seen = look(); };
    auto dq_begin = [&](const int u) {                                // sums of tile u so far
        if (!chained) {
            dqa = zero;
            return;
        }
        if (avail <= u) {
            avail = __builtin_amdgcn_readfirstlane(seen);
            for (int spins = 0; avail <= u;) {
                __builtin_amdgcn_s_sleep(2);
                avail = __builtin_amdgcn_readfirstlane(look());
                if (++spins > MAX_SPINS) { avail = 0x7fffffff; lost = true; }
            }
            asm volatile("" ::: "memory");                            // the sums are read behind the count
        }
        const auto d = __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(reinterpret_cast<const bf16_t *>(part)), 0, TILE_BYTES, 0x00027000);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(d, part_off, 1024 * i, SC1);
#pragma unroll
            for (int e = 0; e < 4; ++e) dqa[4 * i + e] = __builtin_bit_cast(float, (unsigned)w[e]);
        }
        if (lost) dqa = zero + __builtin_nanf("");
    };
    const float oscale = p.scale * cb;                                // dQ and dK carry the factor `scale`; their sums are over dS / cb
    auto dq_end = [&](const int u) {
        if (!last_of_chain) {
            const auto d = __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(reinterpret_cast<const bf16_t *>(part)), 0, TILE_BYTES, 0x00027000);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const f32x4 w = {dqa[4 * i], dqa[4 * i + 1], dqa[4 * i + 2], dqa[4 * i + 3]};
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, w), d, part_off, 1024 * i, SC1);
            }
        } else {
            const int rows = p.L_q - u * BN < BN ? p.L_q - u * BN : BN;
            const int bytes = __builtin_amdgcn_readfirstlane(rows * (int)row_stride * 2);
            const auto d = __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(p.dq + base_q + (size_t)u * BN * row_stride), 0, bytes, 0x00027000);
            const int l = fresh_lane(), qp = l & 31;
            const int row = 32 * nbq + 16 * (qp >> 4) + 8 * ((qp >> 2) & 1) + 4 * ((qp >> 3) & 1) + (qp & 3);
            const bool ok = u * BN + row < nq;
            const int off = (int)(((unsigned)row * (unsigned)row_stride + 32u * dh + 16u * (l >> 5)) * 2u);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                u32x4 w;
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = ok ? pack_bf16(dqa[8 * i + 2 * e] * oscale, dqa[8 * i + 2 * e + 1] * oscale) : 0u;
                __builtin_amdgcn_raw_buffer_store_b128(w, d, off, 16 * i, 0);
            }
        }
        part += 2 * TILE_BYTES;
    };
    auto dq_flag = [&](const int u) {
        if (last_of_chain) return;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (fresh_lane() == 0) __hip_atomic_store(my_flag, u + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    auto dq_fetch_a = [&](auto k_) { qa = lds_read_rows(kt + 16 * decltype(k_)::value); };
    auto dq_fetch_b = [&](auto k_) {
        constexpr int K = decltype(k_)::value;
        const bf16_t *a = reinterpret_cast<const bf16_t *>(smem + dsr0 + 2048 * K);
        const bf16_t *b = reinterpret_cast<const bf16_t *>(smem + dsr1 + 2048 * K);
        qb = lds_read_tr(a, b);
    };

    // operand J of the step on block nb of the tile in `slot`
    auto fetch = [&](auto J_, auto slot, auto nb_c) -> bf16x8 {
        constexpr int J = decltype(J_)::value;
        constexpr int sstep = J / SLOTS, jj = J % SLOTS;
        constexpr int blk = decltype(nb_c)::value + sstep + (jj < 8 ? -1 : 1) + 2;
        constexpr int tile = blk / 2 - 1, brow = (blk % 2) * 32;
        int s = slot.get() + tile + RING_TILES;
        s = s % RING_TILES;
        const int row = s * BN + brow;
        if constexpr (jj < 8) {
            constexpr int half = jj / 4, which = (jj % 4) / 2, mb = jj % 2;
            const bf16_t *a = tr + (row + 16 * half) * LD + 32 * mb + (which == 0 ? Y2 : 0);
            return lds_read_tr(a, a + 8 * LD);
        } else {
            constexpr int which = (jj - 8) / 4, ks = jj % 4;
            return lds_read_rows(rd + row * LD + 16 * ks + (which == 0 ? 0 : Y2));
        }
    };

    constexpr int OPU = 14, UNITS = 8;
    // DQ_PART: 0 none, 1 = first half of the contraction over keys, 2 = second half
    auto step = [&](auto has_prev_c, auto has_next_c, auto drain_c, auto nb_c, auto slot, auto dq_c, auto store_c, const int store_slot) {
        constexpr bool HAS_PREV = decltype(has_prev_c)::value, HAS_NEXT = decltype(has_next_c)::value, DRAIN = decltype(drain_c)::value;
        constexpr int nb = decltype(nb_c)::value, DQP = decltype(dq_c)::value;
        constexpr bool STORE = decltype(store_c)::value;
        constexpr int PAR = nb & 1;
        constexpr ValuOrder<UNITS, OPU, 2, 6> order{};
        constexpr int LEN = DRAIN ? 0 : UNITS * OPU;
        float pv[UNITS][2];
        static_for<0, SLOTS>([&](auto k_) {
            constexpr int k = decltype(k_)::value;
            if constexpr (!DRAIN) {
                constexpr int QUARTER = 2 * nb + (k >= SLOTS / 2);
                if constexpr (k == 0 || k == SLOTS / 2) __builtin_amdgcn_s_setprio(3 - QUARTER);
            }
            if constexpr (STORE && k == 9) {
                store_tile(store_slot);
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (HAS_PREV && (k == 1 || k == 3)) {           // dS of the block before
                constexpr int A = k / 2;
                const int a = dsw ^ (64 * (PAR ^ 1) + 32 * A);
                *reinterpret_cast<u32x4 *>(smem + a) = dsbuf[PAR ^ 1][A];
            }
            if constexpr (k < 8) {
                if constexpr (HAS_PREV) {
                    constexpr int half = k / 4, which = (k % 4) / 2, mb = k % 2;
                    const bf16x8 a = ring[k % RING];
                    if constexpr (which == 0) acc1[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, __builtin_bit_cast(bf16x8, pbuf[PAR ^ 1][half]), acc1[mb], 0, 0, 0);
                    else acc0[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, __builtin_bit_cast(bf16x8, dsbuf[PAR ^ 1][half]), acc0[mb], 0, 0, 0);
                }
            } else if constexpr (HAS_NEXT && !DRAIN) {
                constexpr int which = (k - 8) / 4, ks = k % 4;
                if constexpr (which == 0) sbuf[PAR ^ 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[k % RING], xa[ks], ks == 0 ? zero : sbuf[PAR ^ 1], 0, 0, 0);
                else dbuf[PAR ^ 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[k % RING], xb[ks], ks == 0 ? zero : dbuf[PAR ^ 1], 0, 0, 0);
            }
            constexpr int ahead = k + RING - 1;
            constexpr bool wanted = ahead < 8 ? HAS_PREV : (ahead < SLOTS ? (HAS_NEXT && !DRAIN) : !DRAIN);
            if constexpr (wanted) ring[ahead % RING] = fetch(IntC<ahead>{}, slot, nb_c);
            if constexpr (DQP != 0) {                                 // a dQ contraction every second slot
                if constexpr (k % 2 == 0) {
                    constexpr int K = 8 * (DQP - 1) + k / 2;
                    if constexpr (K == 0) { dq_fetch_a(IntC<0>{}); dq_fetch_b(IntC<0>{}); }
                } else {
                    constexpr int K = 8 * (DQP - 1) + k / 2;
                    dqa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qa, qb, dqa, 0, 0, 0);
                    if constexpr (K + 1 < 16) { dq_fetch_a(IntC<K + 1>{}); dq_fetch_b(IntC<K + 1>{}); }
                }
            }
            static_for<(k * LEN) / SLOTS, ((k + 1) * LEN) / SLOTS>([&](auto i_) {
                constexpr int i = decltype(i_)::value;
                constexpr int w = order.unit[i], o = order.op[i];
                constexpr int ra = 2 * w, rb = 2 * w + 1;
                f32x16 &s = sbuf[PAR];
                f32x16 &dp = dbuf[PAR];
                if constexpr (o == 0) s[ra] = __builtin_amdgcn_exp2f(s[ra]);
                else if constexpr (o == 1) s[rb] = __builtin_amdgcn_exp2f(s[rb]);
                else if constexpr (o == 2) pv[w][0] = __builtin_fmaf(cb, s[ra], 1.0f);
                else if constexpr (o == 3) pv[w][1] = __builtin_fmaf(cb, s[rb], 1.0f);
                else if constexpr (o == 4) pv[w][0] = __builtin_amdgcn_rcpf(pv[w][0]);
                else if constexpr (o == 5) pv[w][1] = __builtin_amdgcn_rcpf(pv[w][1]);
                else if constexpr (o == 6) s[ra] = mul_zero_wins(s[ra], pv[w][0]);
                else if constexpr (o == 7) s[rb] = mul_zero_wins(s[rb], pv[w][1]);
                else if constexpr (o == 8) dp[ra] = pv[w][0] * dp[ra];
                else if constexpr (o == 9) dp[rb] = pv[w][1] * dp[rb];
                else if constexpr (o == 10) dp[ra] = s[ra] * dp[ra];
                else if constexpr (o == 11) dp[rb] = s[rb] * dp[rb];
                else if constexpr (o == 12) dsbuf[PAR][w / 4][w % 4] = pack_bf16(dp[ra], dp[rb]);
                else pbuf[PAR][w / 4][w % 4] = pack_bf16(pv[w][0], pv[w][1]);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    using T_ = IntC<1>;
    using F_ = IntC<0>;
    // ---- prologue: the owner rows are requested, by whole rows, and the second tile.  K and V pass through the place of dS:
    // from there every wave takes its operands, and K^T is made with the transposing read.  (Operands loaded straight from
    // memory and K^T written element by element: 2000 clocks more.)
    {
        const int rows = nk - m0 < BM ? nk - m0 : BM;
        const int bytes = __builtin_amdgcn_readfirstlane(rows * (int)row_stride * 2), pass = 64 * (int)row_stride * 2;
        const auto d1 = __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(p.k + base_k + (size_t)m0 * row_stride), 0, bytes, 0x00027000);
        const auto d2 = __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(p.v + base_k + (size_t)m0 * row_stride), 0, bytes, 0x00027000);
        u32x4 rk[4], rv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) rk[i] = __builtin_amdgcn_raw_buffer_load_b128(d1, (int)ld_off0, i * pass, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) rv[i] = __builtin_amdgcn_raw_buffer_load_b128(d2, (int)ld_off0, i * pass, 0);
        load_tile();
        __builtin_amdgcn_sched_barrier(0);
        *reinterpret_cast<u32x4 *>(w1) = f1;
        *reinterpret_cast<u32x4 *>(w1 + Y2) = f2;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            unsigned char *const home = smem + ds_base + (r0 + 64 * i) * 128 + ((2 * col0) ^ swz(r0));
            *reinterpret_cast<u32x4 *>(home) = rk[i];
            *reinterpret_cast<u32x4 *>(home + DS_BYTES) = rv[i];
        }
    }
    barrier();
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        const unsigned char *const a = smem + ds_base + key * 128 + ((32 * ks + 16 * g) ^ swz(key));
        xa[ks] = *reinterpret_cast<const bf16x8 *>(a);
        xb[ks] = *reinterpret_cast<const bf16x8 *>(a + DS_BYTES);
    }
    // K^T of the wave's keys.  Row position of head-dim column d: 8 (d % 16 / 4) + 4 (d / 16 % 2) + d % 4 of its 32, so that a
    // lane's 16 sums of dQ are 16 columns in a row.
#pragma unroll
    for (int kh = 0; kh < 2; ++kh)                                   // 16 keys
#pragma unroll
        for (int db = 0; db < 4; ++db) {                             // 16 columns
            const int from = wave * 32 + 16 * kh + 4 * (lane >> 4) + (i16 >> 2);
            const s16x4 t = __builtin_amdgcn_ds_read_tr16_b64_v4i16(SIGATTN_LDS_PTR(s16x4, smem + ds_base + from * 128 + ((32 * db + 8 * (i16 & 3)) ^ swz(from))));
            const int pos = 32 * (db / 2) + 8 * (i16 >> 2) + 4 * (db & 1) + (i16 & 3);
            *reinterpret_cast<s16x4 *>(kts + pos * LDT + wave * 32 + 16 * kh + 4 * (lane >> 4)) = t;
        }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) xa[ks] = scale_bf16x8(xa[ks], c1);
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) { acc0[mb] = zero; acc1[mb] = zero; }
    barrier();
    if (m0 + BM > nk) {                                              // rows of dS of the keys behind the end: zeros
        if (!key_ok) {
            const u32x4 z4 = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                *reinterpret_cast<u32x4 *>(smem + ds_base + key * 128 + 64 * g + 16 * i) = z4;
                *reinterpret_cast<u32x4 *>(smem + ds_base + (int)DS_BYTES + key * 128 + 64 * g + 16 * i) = z4;
            }
        }
    }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        sbuf[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_read_rows(rd + 16 * ks), xa[ks], ks == 0 ? zero : sbuf[0], 0, 0, 0);
        dbuf[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_read_rows(rd + Y2 + 16 * ks), xb[ks], ks == 0 ? zero : dbuf[0], 0, 0, 0);
    }

    const int L = ntiles - 1;
    const int tail = nq - L * BN;
    auto mask_block = [&](auto nb_c) {
        constexpr int nb = decltype(nb_c)::value, PAR = nb & 1;
        const short valid = (short)(tail - 32 * nb - 4 * (fresh_lane() >> 5));
        const s16x2 limit = {valid, valid};
#pragma unroll
        for (int w = 0; w < 8; ++w) {
            const short row = (short)(8 * (w / 2) + 2 * (w % 2));
            const s16x2 rows = {row, (short)(row + 1)};
            const unsigned keep = __builtin_bit_cast(unsigned, (s16x2)((rows - limit) >> 15));
            pbuf[PAR][w / 4][w % 4] &= keep;
            dsbuf[PAR][w / 4][w % 4] &= keep;
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto dq_bulk = [&](auto k0, auto k1) {                           // without anything else between: four operand pairs ahead
        constexpr int A = decltype(k0)::value, N = decltype(k1)::value - A;
        bf16x8 a[4], b[4];
        auto get = [&](auto k_) {
            constexpr int K = decltype(k_)::value;
            dq_fetch_a(IntC<A + K>{});
            dq_fetch_b(IntC<A + K>{});
            a[K % 4] = qa;
            b[K % 4] = qb;
        };
        static_for<0, 4>([&](auto k_) { get(k_); });
        __builtin_amdgcn_sched_barrier(0);
        static_for<0, N>([&](auto k_) {
            constexpr int K = decltype(k_)::value;
            dqa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[K % 4], b[K % 4], dqa, 0, 0, 0);
            if constexpr (K + 4 < N) get(IntC<K + 4>{});
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // ON: this wave works on dQ of tile t - 1 (in the second step here and the first step of the next tile)
    int fl = flip;
    auto tile_body = [&](auto slot_c, auto on_c, const int t) {
        constexpr int slot = decltype(slot_c)::value;
        constexpr bool ON = decltype(on_c)::value;
        if constexpr (ON) dq_begin(t - 1);
        step(T_{}, T_{}, F_{}, IntC<0>{}, slot_c, IntC<ON ? 0 : 2>{}, T_{}, (slot + 1) % RING_TILES);
        barrier();
        dsw += fl;
        fl = -fl;
        load_tile();
        if constexpr (!ON) {
            dq_look();
            if (t >= 2) dq_end(t - 2);
        }
        step(T_{}, T_{}, F_{}, IntC<1>{}, slot_c, IntC<ON ? 1 : 0>{}, F_{}, 0);
        if constexpr (!ON) {
            if (t >= 2) dq_flag(t - 2);
        }
    };
    const bool on = ((L - 1) & 1) == grp;                            // at the last tile
    // A wave whose keys are all behind the end moves its share of the tiles and makes its blocks of dQ, and nothing else: the
    // SIMD's other wave has the time (32 x 32 heads of 384 rows 201 -> 185 us; 43 x 12 of up to 700, lognormal 120 -> 103; 86 x 12 of up to
    // 1024 300 -> 288).
    if (m0 + wave * 32 >= nk) {
        for (int t = 0; t < L; ++t) {
            const bool mine = t > 0 && ((t - 1) & 1) == grp;         // dQ of tile t - 1, else (from tile 2 on) of t - 2
            if (mine) dq_begin(t - 1);
            else if (t >= 2) dq_bulk(IntC<8>{}, IntC<16>{});
            store_tile((t + 1) % RING_TILES);
            barrier();
            load_tile();
            if (mine) {
                dq_bulk(IntC<0>{}, IntC<8>{});
            } else if (t > 0) {
                dq_look();
                if (t >= 2) {
                    dq_end(t - 2);
                    dq_flag(t - 2);
                }
            }
        }
        if (L > 0 && on) dq_begin(L - 1);
        if (!on && L >= 2) dq_bulk(IntC<8>{}, IntC<16>{});
        barrier();
        if (!on && L >= 2) {
            dq_end(L - 2);
            dq_flag(L - 2);
        }
        if (on && L > 0) {
            dq_bulk(IntC<0>{}, IntC<16>{});
            dq_end(L - 1);
        }
        if (!on) dq_begin(L);
    } else {
        int slot_rt = 0;
        if (L > 0) {
            step(F_{}, T_{}, F_{}, IntC<0>{}, IntC<0>{}, IntC<0>{}, T_{}, 1);
            barrier();
            load_tile();
            step(T_{}, T_{}, F_{}, IntC<1>{}, IntC<0>{}, IntC<0>{}, F_{}, 0);
            int t = 1, state = grp ? 3 : 0;
            while (t < L) {
                if (state == 0) { tile_body(IntC<1>{}, T_{}, t); state = 1; ++t; }
                if (t < L && state == 1) { tile_body(IntC<2>{}, F_{}, t); state = 2; ++t; }
                if (t < L && state == 2) { tile_body(IntC<0>{}, T_{}, t); state = 3; ++t; }
                if (t < L && state == 3) { tile_body(IntC<1>{}, F_{}, t); state = 4; ++t; }
                if (t < L && state == 4) { tile_body(IntC<2>{}, T_{}, t); state = 5; ++t; }
                if (t < L && state == 5) { tile_body(IntC<0>{}, F_{}, t); state = 0; ++t; }
            }
            slot_rt = L % RING_TILES;
            if (on) {
                dq_begin(L - 1);
            }
            step(T_{}, T_{}, F_{}, IntC<0>{}, DynInt{slot_rt}, IntC<0>{}, F_{}, 0);
            if (!on && L >= 2) dq_bulk(IntC<8>{}, IntC<16>{});
        } else {
            step(F_{}, T_{}, F_{}, IntC<0>{}, DynInt{0}, IntC<0>{}, F_{}, 0);
        }
        if (tail < BN) mask_block(IntC<0>{});
        barrier();
        if (L > 0) dsw += fl;
        if (!on && L >= 2) dq_end(L - 2);
        step(T_{}, F_{}, F_{}, IntC<1>{}, DynInt{slot_rt}, IntC<0>{}, F_{}, 0);
        if (tail < BN) mask_block(IntC<1>{});
        if (!on && L >= 2) dq_flag(L - 2);
        if (on && L > 0) dq_bulk(IntC<0>{}, IntC<16>{});
        step(T_{}, F_{}, T_{}, IntC<0>{}, DynInt{(slot_rt + 1) % RING_TILES}, IntC<0>{}, F_{}, 0);
        if (on && L > 0) dq_end(L - 1);
        if (!on) dq_begin(L);
    }
    barrier();
    if (on) {
        if (L > 0) dq_flag(L - 1);
    } else {
        dq_bulk(IntC<0>{}, IntC<16>{});
        dq_end(L);
        dq_flag(L);
    }

    // ---- dK, dV
    auto chunk = [&](const f32x16 &a, const int pr, const float f) {   // columns of q4 = 2 pr + g
        const unsigned e0 = pack_bf16(a[8 * pr + 0] * f, a[8 * pr + 1] * f), e1 = pack_bf16(a[8 * pr + 2] * f, a[8 * pr + 3] * f);
        const unsigned o0 = pack_bf16(a[8 * pr + 4] * f, a[8 * pr + 5] * f), o1 = pack_bf16(a[8 * pr + 6] * f, a[8 * pr + 7] * f);
        const auto s0 = __builtin_amdgcn_permlane32_swap(e0, o0, false, false);
        const auto s1 = __builtin_amdgcn_permlane32_swap(e1, o1, false, false);
        const u32x4 w = {s0[0], s1[0], s0[1], s1[1]};
        return w;
    };
    {
        const int rows = p.L_k - m0 < BM ? p.L_k - m0 : BM;
        const int bytes = __builtin_amdgcn_readfirstlane(rows * (int)row_stride * 2);
        const size_t base = base_k + (size_t)m0 * row_stride;
        const auto d0 = __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(p.dk + base), 0, bytes, 0x00027000);
        const auto d1 = __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(p.dv + base), 0, bytes, 0x00027000);
        const int l = fresh_lane(), row = wave * 32 + (l & 31);
        const bool ok = m0 + row < nk;
        const int off = (int)(((unsigned)row * (unsigned)row_stride + 8u * (l >> 5)) * 2u);
        const u32x4 z4 = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int pr = 0; pr < 2; ++pr) {
                const u32x4 a = chunk(acc0[mb], pr, oscale), b = chunk(acc1[mb], pr, 1.0f);
                __builtin_amdgcn_raw_buffer_store_b128(ok ? a : z4, d0, off + 2 * (32 * mb + 16 * pr), 0, 0);
                __builtin_amdgcn_raw_buffer_store_b128(ok ? b : z4, d1, off + 2 * (32 * mb + 16 * pr), 0, 0);
            }
    }
    zero_dq_share();
}

}  // namespace onepass
}  // namespace sigattn
