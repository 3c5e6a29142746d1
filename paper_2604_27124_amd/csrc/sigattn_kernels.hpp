// Device code for padded bidirectional sigmoid attention on gfx950 (CDNA4).
//
// One kernel template serves the three passes of the method (paper appendix Alg. 1-3):
//
//   FWD   (Alg. 1): owner = a tile of queries,  streamed = key/value tiles.   Out = O
//   DQ    (Alg. 2): owner = a tile of queries,  streamed = key/value tiles.   Out = dQ
//   DKDV  (Alg. 3): owner = a tile of keys,     streamed = query/dO tiles.    Out = dK, dV
//
// "Owner" rows are held in registers for the whole kernel as MFMA B operands; "streamed" tiles go
// HBM -> registers -> LDS (a ring of four tiles) and are read from LDS as MFMA A operands, either row-wise
// (contraction over the head dimension) or through the transposing LDS read (contraction over tokens).
// Every score tile is computed transposed, streamed x owner, so that the fp32 accumulator of one lane
// holds one owner column and several streamed rows: after the fused sigmoid those registers are, without
// any shuffle, the bf16 B operand of the next contraction over streamed tokens.
//
// The inner loop is a software pipeline over 32-row blocks of the streamed tensors.  One step holds, for
// block b, the score contractions of block b + 1, the sigmoid of block b and the output contractions of
// block b - 1.  A step is cut into slots of one MFMA each; every slot also carries an equal share of the
// step's VALU work and, at most, the LDS read of one later A operand.  A operands travel through a small
// ring of registers and are requested RING - 1 operands before their first use, so that no MFMA waits for
// the LDS.  The order inside a step is pinned with scheduling fences; nothing is left to reorder.
//
// v_mfma_f32_32x32x16_bf16 operand layout used below (lane l, c = l % 32, g = l / 32):
//   A[32 x 16]: lane holds row c,    k = 8 g + 0..7
//   B[16 x 32]: lane holds column c, k = 8 g + 0..7
//   C[32 x 32]: lane holds column c, register i holds row 8 (i / 4) + 4 g + (i % 4)
// ds_read_b64_tr_b16 within a group of 16 lanes: destination lane i, element e comes from the 8 bytes
// addressed by lane (i / 4 + 4 e), 16-bit column (i % 4).  With lane r of the group pointing at
// (row r / 4, column 4 (r % 4)) of a row-major [4 x 16] block, lane i receives column i, rows 0..3.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sigattn {

typedef __bf16 bf16_t;
typedef bf16_t bf16x8 __attribute__((ext_vector_type(8)));
typedef bf16_t bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

enum Mode { FWD = 0, DQ = 1, DKDV = 2 };

template <int V>
struct IntC {
    static constexpr int value = V;
    __device__ __forceinline__ constexpr int get() const { return V; }
};
struct DynInt {   // same interface as IntC for a value only known at run time
    int v;
    __device__ __forceinline__ int get() const { return v; }
};

template <int I, int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (I < N) {
        f(IntC<I>{});
        static_for<I + 1, N>(f);
    }
}

// Owner side = the tensors whose rows a workgroup keeps (queries in FWD and DQ, keys in DKDV); streamed side
// = the other one.  The two sides have padded lengths and valid lengths of their own (appendix Alg. 1-3:
// L_q, L_k, n_q, n_k); self-attention passes the same numbers twice.
struct Params {
    const bf16_t *q, *k, *v, *d_o;   // inputs: q, d_o [B, L_q, H, D];  k, v [B, L_k, H, D]
    bf16_t *out0;                    // FWD: O;  DQ: dQ;  DKDV: dK
    bf16_t *out1;                    // DKDV: dV
    const int32_t *seqlens;          // [B] valid lengths of the owner side
    const int32_t *seqlens_str;      // [B] valid lengths of the streamed side
    const float *bias;               // [B]
    float scale;
    int B, N, H;                     // N: padded length of the owner side
    int N_str;                       // padded length of the streamed side
    int in_order;                    // work mapping: 1 = batch order, 0 = longest sequences first
    int groups;                      // batch order: 0 = a workgroup per owner tile, else this many for the owner tiles of
                                     // a sequence, and `wide_groups` for those of each of the first `wide_seqs`
    int wide_groups, wide_seqs;
    float *db_part;                  // DQ with bias gradient: one partial sum per owner tile, [B][H][tiles of a sequence]
};

#define SIGATTN_LDS_PTR(T, p) ((__attribute__((address_space(3))) T *)(p))

__device__ __forceinline__ bf16x8 lds_read_rows(const bf16_t *p) {
    return *reinterpret_cast<const bf16x8 *>(p);
}

// Two transposing reads -> the 8 contraction slots of one A operand.
__device__ __forceinline__ bf16x8 lds_read_tr(const bf16_t *p_lo, const bf16_t *p_hi) {
    s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(SIGATTN_LDS_PTR(s16x4, p_lo));
    s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(SIGATTN_LDS_PTR(s16x4, p_hi));
    s16x8 r = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, r);
}

// a * b under the rule 0 * x = 0 for every x, also +-inf and NaN (v_mul_legacy_f32).
__device__ __forceinline__ float mul_zero_wins(float a, float b) {
    float r;
    asm("v_mul_legacy_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

__device__ __forceinline__ unsigned pack_bf16(float a, float b) {
    f32x2 f = {a, b};
    bf16x2 h = __builtin_convertvector(f, bf16x2);   // v_cvt_pk_bf16_f32, round to nearest even
    return __builtin_bit_cast(unsigned, h);
}

// Shape of one pipeline step and of the two instruction streams that are woven into it.
template <int MODE, int D, int QB, int NW, int BN, int LD1, int LD2, int RING>
struct Cfg {
    static constexpr bool HAS2 = (MODE != FWD);    // a second owner tensor and a second score tile (dP)
    static constexpr int BM = NW * 32 * QB;        // owner rows per workgroup
    static constexpr int THREADS = NW * 64;
    static constexpr int KS = D / 16;              // MFMA steps over the head dimension
    static constexpr int MB = D / 32;              // 32-row blocks of a transposed [D x 32] output
    static constexpr int NB = BN / 32;             // 32-row blocks of a streamed tile
    static constexpr int CH = D / 8;               // 16-byte chunks per row
    static constexpr int PER = (BN * CH) / THREADS;  // chunks per thread per streamed tensor
    static constexpr int NBUF = 4;                 // LDS ring: tile t lives in slot t % 4
    static constexpr size_t LDS_BYTES = (size_t)NBUF * BN * (LD1 + LD2) * sizeof(bf16_t);
    // A operands of one step, in the order they are used: first the row-wise ones of the score
    // contractions (block b + 1), then the transposed ones of the output contractions (block b - 1).
    static constexpr int NT = HAS2 ? 2 : 1;        // score tiles per block (S, dP)
    static constexpr int NO = (MODE == DKDV) ? 2 : 1;   // output tensors
    static constexpr int NA = KS * NT;
    static constexpr int NC = 2 * MB * NO;
    static constexpr int NOPS = NA + NC;
    static constexpr int SLOTS = NOPS * QB;        // one MFMA per slot
    // VALU work: units of two score elements (one packed bf16 register of the next B operand).
    static constexpr int UNITS = QB * 8;
    // LDS placement of a streamed row t: element offset t * LD + lds_shift(t).  Mode 0 is the plain padded
    // layout (row stride 16 bytes modulo 32): conflict-free for the 16-byte row-wise reads of 16 consecutive
    // rows.  The transposing 8-byte reads of a half-wave touch four consecutive rows; at D = 64 that layout
    // costs them nothing measurable, at D = 128 (272-byte rows) it quarters their rate.  Mode 2, for D = 128
    // tensors that are read transposed: 288-byte rows (32 bytes modulo the 256 bytes of the banks), the 32
    // output rows of one MFMA taken as two groups of 16 head-dim columns that lie 128 bytes apart, so that
    // the four rows of a read fall into disjoint banks; every second group of eight rows is shifted by a
    // further 16 bytes, which keeps the row-wise reads conflict-free under that stride.
    static constexpr int lds_mode(int LD) { return ((2 * LD) % 256 == 32 && D == 128) ? 2 : 0; }
    static constexpr int LM1 = lds_mode(LD1), LM2 = lds_mode(LD2);
    static_assert(LM1 != 2 || LD1 >= D + 8, "mode 2 shifts a row by up to 16 bytes");
    static_assert(LM2 != 2 || LD2 >= D + 8, "mode 2 shifts a row by up to 16 bytes");
    static_assert((BN * CH) % THREADS == 0, "tile does not split evenly over the workgroup");
    // Two blocks, not any even number: once the last tile's first block has been through, no score contraction reads the
    // owner rows any more, and those of the next owner tile are requested into their registers.
    static_assert(D % 32 == 0 && NB == 2, "tile shape (two 32-row blocks per streamed tile)");
    static_assert(LD1 % 8 == 0 && LD2 % 8 == 0 && LD1 >= D && LD2 >= D, "LDS row stride");
    static_assert((NB * NOPS) % RING == 0 && RING >= 2 && RING <= NOPS, "operand ring does not close over a tile");
};

// Element offset added to row `row` of a streamed tile in LDS (see Cfg::lds_mode), the extra offset of the
// second transposing read (eight rows further on), and the column layout of the transposed operand.
template <int LM>
__device__ __forceinline__ constexpr int lds_shift(int row) {
    return LM == 2 ? 8 * ((row >> 3) & 1) : 0;
}
template <int LM>
struct TrLayout {
    static constexpr int HI_EXTRA = LM == 2 ? 8 : 0;                    // lds_shift(row + 8) - lds_shift(row), row % 8 < 4
    static constexpr int GROUP_COLS = LM == 2 ? 64 : 16;                // column distance of the two 16-lane groups
    static constexpr int MB_COLS = LM == 2 ? 16 : 32;                   // column step from one output block to the next
    // head-dim column of accumulator registers 4 q4 .. 4 q4 + 3 of output block mb (without the 4 g of the lane)
    static constexpr int out_col(int mb, int q4) {
        return LM == 2 ? 16 * mb + 64 * (q4 >> 1) + 8 * (q4 & 1) : 32 * mb + 8 * q4;
    }
};

// The VALU instructions of one step as a flat list.  Each unit (two score elements) runs through three
// stages -- exponentials | denominator and reciprocal | products and packing -- and the list is skewed by
// one unit per stage, so that an instruction never follows directly on the one that feeds it.
template <int UNITS, int OPU, int S0, int S1>
struct ValuOrder {
    static constexpr int LEN = UNITS * OPU;
    int unit[LEN];
    int op[LEN];
    constexpr ValuOrder() : unit{}, op{} {
        int n = 0;
        for (int tau = 0; tau < UNITS + 2; ++tau) {
            if (tau < UNITS)
                for (int o = 0; o < S0; ++o) { unit[n] = tau; op[n] = o; ++n; }
            if (tau >= 1 && tau - 1 < UNITS)
                for (int o = S0; o < S1; ++o) { unit[n] = tau - 1; op[n] = o; ++n; }
            if (tau >= 2 && tau - 2 < UNITS)
                for (int o = S1; o < OPU; ++o) { unit[n] = tau - 2; op[n] = o; ++n; }
        }
    }
};

// Write zeros over owner rows [row0, row1) of one (z, h) slice of `out`.
template <int D, int THREADS>
__device__ __forceinline__ void zero_rows(bf16_t *out, size_t slice_base, size_t row_stride, int row0, int row1) {
    constexpr int CH = D / 8;
    const int total = (row1 - row0) * CH;
    const u32x4 z = {0u, 0u, 0u, 0u};
    for (int c = threadIdx.x; c < total; c += THREADS) {
        const int r = row0 + c / CH;
        *reinterpret_cast<u32x4 *>(out + slice_base + (size_t)r * row_stride + (size_t)(c % CH) * 8) = z;
    }
}

// bf16 x 8 times a float, rounded back to bf16 (used once per kernel, on the owner rows).
__device__ __forceinline__ bf16x8 scale_bf16x8(const bf16x8 v, const float f) {
    u32x4 r;
#pragma unroll
    for (int j = 0; j < 4; ++j) r[j] = pack_bf16((float)v[2 * j] * f, (float)v[2 * j + 1] * f);
    return __builtin_bit_cast(bf16x8, r);
}

// Longest-first work mapping.  The launch is a 1-D grid with one workgroup per owner tile of every
// (z, h); hardware hands consecutive workgroup ids to the 8 XCDs round-robin and to free CUs in order.
// Ids are therefore mapped so that the tiles of the LONGEST sequences come first (their cost is
// proportional to the sequence's valid length), every XCD receives every 8th id of that sorted list, and
// within one sequence the ids of one XCD are consecutive tiles of the same head; wholly padded tiles,
// which only write zeros, come last.  Sequences are ranked inside the kernel from seqlens, so the host
// never needs the lengths.  Ties keep batch order.  Where workgroups are short and many the ranking costs more
// than the order gives, and the host asks for batch order instead (see batch_order() on the host side).
// The ranking has two forms, by its cost per workgroup:
//   up to MAP_WAVE_B sequences: every wave ranks them for itself in registers, one sequence per lane, by exact
//       length -- one load, no LDS, no barrier;
//   larger batches: by their number of owner tiles (at most MAP_CLASSES of them), with a histogram and
//       block-wide prefix sums (work per thread grows with B / THREADS, not with B).
constexpr int MAP_WAVE_B = 64;
constexpr int MAP_CLASSES = 1024;

// Ids [lo, lo + cnt) are the H * tiles valid ids of one sequence.  Hardware deals consecutive ids round-robin
// to the 8 XCDs, each with an L2 of its own; the ids of the range that land on one XCD take consecutive
// tiles of one head (then of the next), so a head's streamed slab is fetched by one or two XCDs only.
// Returns the position of `id` in that XCD-major order of the range.
__device__ __forceinline__ int xcd_major_index(int id, int lo, int cnt) {
    const int idx = id - lo, x = id & 7;
    int e = 0;                                      // ids of this range on XCDs below x
    for (int y = 0; y < x; ++y) {
        const int first = (y - lo) & 7;             // first index of the range that lands on XCD y
        e += (first < cnt) ? ((cnt - first + 7) >> 3) : 0;
    }
    return e + ((idx - ((x - lo) & 7)) >> 3);       // plus the position among the ids on XCD x
}

struct MapScratch {                       // LDS of the ranking (more than MAP_WAVE_B sequences)
    int res[4];                           // z, n, h, m0 of this workgroup
    int hist[MAP_CLASSES];                // owner tiles per class
    int wave[16];                         // wave totals of a block-wide prefix sum
    int pick[4];                          // class holding this id (-1: padded part) | tiles before it | all valid tiles | found
};

// What one workgroup does: `count` owner tiles of one sequence, starting with the tile at row m0 of head h and going on
// through the valid tiles of that head and of the heads behind it.  shares = 0: the tile alone, which may be padding.
// Else the workgroup also writes its share of the zeros behind the sequence's valid tiles.
struct Work { int z, n, h, m0, count, share, shares; };

// Batch order: position of `id` among the `cnt` ids [lo, lo + cnt) of sequence z, dealt to the XCDs in runs as above.
// Which XCD takes which run turns with the sequence: runs differ in their share of padding, and an XCD keeps the ids
// that hardware deals to it while the others wait for the slowest.
__device__ __forceinline__ int batch_order_pos(const int id, const int lo, const int cnt, const int turn) {
    return (xcd_major_index(id, lo, cnt) + turn % cnt) % cnt;
}

// A workgroup per owner tile: H * T ids per sequence, consecutive tiles of a head in a run.  Where the tiles of a head
// begin turns with the head, since a shader engine gets every fourth id of an XCD's.  (Without this second turn 280 of
// the 512 workgroups that fit were running in a launch of 24576: dK/dV at B = 512, N = 512 took 608 us instead of 488.)
__device__ __forceinline__ void batch_order_tile(const int id, const int H, const int T, int &z, int &h, int &tile) {
    const int cnt = H * T;
    z = id / cnt;
    const int e = batch_order_pos(id, z * cnt, cnt, (z & 7) * ((cnt + 7) >> 3));
    h = e / T;
    tile = (e - h * T + (T >= 4 ? h + z : (h + z) / (4 / T))) % T;
}

// Several owner tiles per workgroup: the last workgroups of a sequence have one tile less, so the turn is by one id more
// than a run.
__device__ __forceinline__ int shared_turn(const int z, const int cnt) {
    return (int)((unsigned)z * (unsigned)(((cnt + 7) >> 3) + 1) % (unsigned)cnt);
}

// The sequence of an id and the ids of that sequence, [lo, lo + cnt).
__device__ __forceinline__ void batch_order_range(const int id, const int wide_seqs, const int wide_groups, const int groups,
                                                  int &z, int &lo, int &cnt) {
    const int wide = wide_seqs * wide_groups;
    const bool w = id < wide;
    const int first = w ? 0 : wide;
    cnt = w ? wide_groups : groups;
    const int k = (id - first) / cnt;
    z = (w ? 0 : wide_seqs) + k;
    lo = first + k * cnt;
}

template <int BM>
__device__ __forceinline__ int owner_tiles(const Params &p) { return (p.N + BM - 1) / BM; }    // per (z, h), padded ones included

__device__ __forceinline__ int owner_length(const Params &p, int b) {
    const int v = p.seqlens[b];
    return v < 0 ? 0 : (v > p.N ? p.N : v);
}

// Workgroup `g` of the `groups` that share the valid owner tiles of sequence z (all heads, tile by tile).
template <int BM>
__device__ __forceinline__ Work batch_order_share(const Params &p, const int z, const int g, const int groups) {
    const int n = owner_length(p, z);
    const int tiles = (n + BM - 1) / BM, jobs = tiles * p.H;
    const int each = jobs / groups, extra = jobs % groups;
    const int first = g * each + (g < extra ? g : extra), count = each + (g < extra ? 1 : 0);
    const int h = count > 0 ? first / tiles : 0;
    return {z, n, h, (first - h * tiles) * BM, count, g, groups};
}

template <int BM, int THREADS>
__device__ __forceinline__ Work map_work(const Params &p, const int id, MapScratch &scratch) {
    static_assert((BM & (BM - 1)) == 0, "owner tile rows: a power of two");
    const int T = owner_tiles<BM>(p);
    int z, h, n, m0;
    int *const s_res = scratch.res;
    auto len_of = [&](int b) { return owner_length(p, b); };
    if (p.groups) {
        int lo, cnt;
        batch_order_range(id, p.wide_seqs, p.wide_groups, p.groups, z, lo, cnt);
        return batch_order_share<BM>(p, z, batch_order_pos(id, lo, cnt, shared_turn(z, cnt)), cnt);
    }
    if (p.in_order) {
        int tile;
        batch_order_tile(id, p.H, T, z, h, tile);
        return {z, len_of(z), h, tile * BM, 1, 0, 0};
    }
    if (p.B <= MAP_WAVE_B) {
        // Id ranges as below: the valid tiles of every sequence, longest first, H ids per tile; then the padded
        // tiles in batch order.  Lane l sums the tiles in front of sequence l, whose length every lane reads from
        // lane u by a scalar read; the lane whose range holds this workgroup's id is found with a ballot.
        const int lane = threadIdx.x & 63;
        const int mine = lane < p.B ? len_of(lane) : 0;
        const int my_tiles = (mine + BM - 1) / BM;
        int before = 0, all_valid = 0;
        for (int u = 0; u < p.B; ++u) {
            const int o = __builtin_amdgcn_readlane(mine, u), tiles = (o + BM - 1) / BM;
            before += (o >= mine + (lane <= u)) ? tiles : 0;        // longer, or as long and earlier in the batch
            all_valid += tiles;
        }
        int lo = before, cnt = my_tiles;
        const bool padded = id >= all_valid * p.H;                  // uniform
        if (padded) {                                               // exclusive prefix sum of the padded tiles
            cnt = lane < p.B ? T - my_tiles : 0;
            int incl = cnt;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int up = __shfl_up(incl, off, 64);
                incl += (lane >= off) ? up : 0;
            }
            lo = all_valid + incl - cnt;
        }
        lo *= p.H;
        const unsigned long long hit = __builtin_amdgcn_ballot_w64(lane < p.B && id >= lo && id < lo + cnt * p.H);
        const int src = __builtin_ctzll(hit);                       // exactly one lane: the ranges tile the grid
        z = src;
        n = __builtin_amdgcn_readlane(mine, src);
        lo = __builtin_amdgcn_readlane(lo, src);
        cnt = __builtin_amdgcn_readlane(cnt, src);
        if (padded) {
            h = (id - lo) % p.H;
            m0 = ((n + BM - 1) / BM + (id - lo) / p.H) * BM;
        } else {
            const int e = xcd_major_index(id, lo, cnt * p.H);
            h = e / cnt;
            m0 = (e % cnt) * BM;
        }
        return {z, n, h, m0, 1, 0, 0};
    }
    // ---- more sequences than lanes.  A sequence's class is its number of owner tiles
    // (class 0 = T tiles, the longest; T <= MAP_CLASSES is the host's rule).
    // Id ranges: classes in ascending order, inside a class the sequences in batch order, H ids per tile;
    // then the padded tiles in batch order.  All positions are kept in tiles: a sequence whose tiles are
    // [tb, tb + tiles) of that list owns the ids [H tb, H (tb + tiles)).
    int *const s_hist = scratch.hist, *const s_wave = scratch.wave, *const s_pick = scratch.pick;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    auto class_of = [&](int tiles) { return T - tiles; };      // tiles in [1, T]
    for (int i = tid; i < MAP_CLASSES; i += THREADS) s_hist[i] = 0;
    if (tid == 0) { s_pick[0] = -1; s_pick[3] = 0; }
    __syncthreads();
    for (int b = tid; b < p.B; b += THREADS) {
        const int tiles = (len_of(b) + BM - 1) / BM;
        if (tiles > 0) atomicAdd(&s_hist[class_of(tiles)], tiles);
    }
    __syncthreads();
    const int tgt = id / p.H;             // position of this id's tile in the list of all tiles
    if (wave == 0) {                      // prefix over the classes: each lane sums a run of them, lanes by shuffles
        constexpr int RUN = MAP_CLASSES / 64;
        int mine = 0;
        for (int i = 0; i < RUN; ++i) mine += s_hist[lane * RUN + i];
        int incl = mine;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int up = __shfl_up(incl, off, 64);
            incl += (lane >= off) ? up : 0;
        }
        if (lane == 63) s_pick[2] = incl;
        int before = incl - mine;
        if (tgt >= before && tgt < incl) {            // at most one lane
            int c = lane * RUN;
            while (tgt >= before + s_hist[c]) { before += s_hist[c]; ++c; }
            s_pick[0] = c; s_pick[1] = before;
        }
    }
    __syncthreads();
    const int cls = s_pick[0], all_valid = s_pick[2];
    const int base = cls >= 0 ? s_pick[1] : all_valid;      // tiles in front of the part that is searched
    const int rest = tgt - base;                            // position inside that part, in batch order
    int running = 0;
    for (int c0 = 0; c0 < p.B; c0 += THREADS) {
        const int b = c0 + tid;
        int len = 0, tiles = 0, v = 0;
        if (b < p.B) {
            len = len_of(b);
            tiles = (len + BM - 1) / BM;
            v = cls >= 0 ? ((tiles > 0 && class_of(tiles) == cls) ? tiles : 0) : T - tiles;
        }
        int incl = v;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int up = __shfl_up(incl, off, 64);
            incl += (lane >= off) ? up : 0;
        }
        if (lane == 63) s_wave[wave] = incl;
        __syncthreads();
        int offset = 0, total = 0;
#pragma unroll
        for (int w = 0; w < THREADS / 64; ++w) {
            const int t = s_wave[w];
            offset += (w < wave) ? t : 0;
            total += t;
        }
        const int hi = running + offset + incl, lo_t = hi - v;
        if (v > 0 && rest >= lo_t && rest < hi) {           // exactly one thread of one chunk
            const int lo = (base + lo_t) * p.H;             // first id of this sequence's range
            if (cls >= 0) {
                const int e = xcd_major_index(id, lo, tiles * p.H);
                s_res[0] = b; s_res[1] = len; s_res[2] = e / tiles; s_res[3] = (e % tiles) * BM;
            } else {
                const int r = id - lo;
                s_res[0] = b; s_res[1] = len; s_res[2] = r % p.H; s_res[3] = (tiles + r / p.H) * BM;
            }
            s_pick[3] = 1;
        }
        __syncthreads();
        if (s_pick[3]) break;
        running += total;
    }
    return {s_res[0], s_res[1], s_res[2], s_res[3], 1, 0, 0};
}

// The lane, worked out anew: what is computed from it is computed again for every owner tile instead of holding
// registers through the main loop, which has none to spare.
__device__ __forceinline__ int fresh_lane() {
    int all = -1;
    asm volatile("" : "+s"(all));
    return __builtin_amdgcn_mbcnt_hi(all, __builtin_amdgcn_mbcnt_lo(all, 0));
}

// A pointer that is the same in all lanes, in scalar registers.
__device__ __forceinline__ bf16_t *uniform_ptr(const bf16_t *p) {
    const unsigned long long a = reinterpret_cast<unsigned long long>(p);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a), hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
    return reinterpret_cast<bf16_t *>((unsigned long long)hi << 32 | lo);
}

// The owner tiles of one workgroup, one pass.  `smem`: Cfg::LDS_BYTES bytes.
template <int MODE, int D, int QB, int NW, int BN, int LD1, int LD2, int RING, bool WITH_DB>
__device__ __forceinline__ void run_pass(const Params &p, const Work work, unsigned char *const smem, float *const s_db) {
    static_assert(!WITH_DB || MODE == DQ, "the bias gradient rides on the dQ kernel");
    using C = Cfg<MODE, D, QB, NW, BN, LD1, LD2, RING>;
    constexpr bool HAS2 = C::HAS2;
    constexpr int Q2 = HAS2 ? QB : 1;
    constexpr int NB = C::NB, NA = C::NA, NOPS = C::NOPS, SLOTS = C::SLOTS, NT = C::NT, NO = C::NO, MB = C::MB;
    constexpr float LOG2E = 1.4426950408889634f;

    bf16_t *y1s = reinterpret_cast<bf16_t *>(smem);                 // [NBUF][BN][LD1]
    bf16_t *y2s = y1s + C::NBUF * BN * LD1;                         // [NBUF][BN][LD2]

    const int z = __builtin_amdgcn_readfirstlane(work.z);      // uniform across the workgroup: keep them in scalar registers
    const int n = __builtin_amdgcn_readfirstlane(work.n);
    int h = __builtin_amdgcn_readfirstlane(work.h);                 // owner tile in hand, and how many are left with it
    int m0 = __builtin_amdgcn_readfirstlane(work.m0);
    int left = __builtin_amdgcn_readfirstlane(work.count);
    const int share = __builtin_amdgcn_readfirstlane(work.share), shares = __builtin_amdgcn_readfirstlane(work.shares);
    const size_t row_stride = (size_t)p.H * D;
    const size_t seq_base = (size_t)z * p.N * row_stride;           // owner side: element offset of row 0 of sequence z
    const size_t seq_base_s = (size_t)z * p.N_str * row_stride;     // streamed side
    int ns = n;                                                     // valid rows of the streamed side
    if (p.seqlens_str != p.seqlens || p.N_str != p.N) {             // self-attention: the mapping already has it
        ns = p.seqlens_str[z];
        ns = ns < 0 ? 0 : (ns > p.N_str ? p.N_str : ns);
    }
    ns = __builtin_amdgcn_readfirstlane(ns);

    const int T = owner_tiles<C::BM>(p);
    auto db_slot = [&](int head, int row) { return ((size_t)z * p.H + head) * T + row / C::BM; };

    // Padding (block-sparse early exit): owner rows in tiles that are wholly padded, or all rows if there is nothing to
    // stream, are zeros and nothing else.
    const int valid_tiles = ns == 0 ? 0 : (n + C::BM - 1) / C::BM;  // per head
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (shares == 0) {
        if (m0 >= n || ns == 0) {
            const int m1 = (m0 + C::BM < p.N) ? m0 + C::BM : p.N;
            zero_rows<D, C::THREADS>(p.out0, seq_base + (size_t)h * D, row_stride, m0, m1);
            if (MODE == DKDV) zero_rows<D, C::THREADS>(p.out1, seq_base + (size_t)h * D, row_stride, m0, m1);
            if (WITH_DB && tid == 0) p.db_part[db_slot(h, m0)] = 0.f;
            return;
        }
    }
    auto zero_share = [&]() {                                       // this workgroup's share of them, all heads together
        if (shares == 0 || valid_tiles == T) return;
        const u32x4 z4 = {0u, 0u, 0u, 0u};
        const int me = share * C::THREADS + wave * 64 + fresh_lane();
        const size_t from = seq_base + (size_t)valid_tiles * C::BM * row_stride;
        const size_t chunks = (size_t)(p.N - valid_tiles * C::BM) * (row_stride / 8);
        for (size_t i = (size_t)me; i < chunks; i += (size_t)shares * C::THREADS) {
            *reinterpret_cast<u32x4 *>(p.out0 + from + i * 8) = z4;
            if (MODE == DKDV) *reinterpret_cast<u32x4 *>(p.out1 + from + i * 8) = z4;
        }
        if (WITH_DB) {
            const int padded = T - valid_tiles;
            for (int i = me; i < padded * p.H; i += shares * C::THREADS)
                p.db_part[db_slot(i / padded, (valid_tiles + i % padded) * C::BM)] = 0.f;
        }
    };
    if (left == 0 || ns == 0) {
        zero_share();
        return;
    }

    const bf16_t *x1 = (MODE == DKDV) ? p.k : p.q;                  // owner tensors
    const bf16_t *x2 = (MODE == DKDV) ? p.v : p.d_o;
    const bf16_t *y1 = (MODE == DKDV) ? p.q : p.k;                  // streamed tensors
    const bf16_t *y2 = (MODE == DKDV) ? p.d_o : p.v;

    const int lane = tid & 63;
    const int c = lane & 31, g = lane >> 5;

    // sigma(x) = 1 / (1 + cb 2^t') with t' = c1 <q, k>, c1 = -scale log2 e, cb = 2^(-bias log2 e).
    // c1 is folded into the owner operand of the score contraction (one extra bf16 rounding of that
    // operand), so t' leaves the MFMA ready for exp2; cb rides on the FMA that forms the denominator.
    // The exponent of cb is clamped to +-126 (|bias| <= 87.3 is exact; beyond that sigma is saturated).
    // cb is finite and non-zero, so cb 2^t' is 0, finite or +inf but never NaN, and P lands in [0, 1].
    const float c1 = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, -p.scale * LOG2E)));
    const float cb = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int,
        __builtin_amdgcn_exp2f(__builtin_fminf(__builtin_fmaxf(-p.bias[z] * LOG2E, -126.0f), 126.0f)))));

    // ---- owner rows -> registers (B operands): lane holds row c of each 32-block, d = 16 ks + 8 g + 0..7.  Read through
    // a buffer descriptor that ends with the sequence's last valid row (see load_tile below): rows behind it are zeros.
    bf16x8 xa[QB][C::KS];
    bf16x8 xb[Q2][HAS2 ? C::KS : 1];
    auto row_offset = [&]() {                                       // bytes from an owner tile's first row to this lane's
        const int l = fresh_lane();
        return ((unsigned)(wave * 32 * QB + (l & 31)) * (unsigned)row_stride + 8u * (l >> 5)) * 2u;
    };
    const int block_bytes = 32 * (int)row_stride * 2;
    auto load_owner = [&](const int head, const int row0) {
        const int rows = n - row0 < C::BM ? n - row0 : C::BM;
        const size_t base = seq_base + (size_t)row0 * row_stride + (size_t)head * D;
        const int bytes = __builtin_amdgcn_readfirstlane(rows * (int)row_stride * 2);
        const auto d1 = __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(x1 + base), 0, bytes, 0x00027000);
        const auto d2 = __builtin_amdgcn_make_buffer_rsrc(uniform_ptr((HAS2 ? x2 : x1) + base), 0, bytes, 0x00027000);
        const int off = (int)row_offset();
        // the rows that are scaled come last: a wait for them is a wait for all
        if (HAS2)
#pragma unroll
            for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                for (int ks = 0; ks < C::KS; ++ks)
                    xb[HAS2 ? qb : 0][HAS2 ? ks : 0] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(d2, off + 32 * ks, qb * block_bytes, 0));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int ks = 0; ks < C::KS; ++ks)
                xa[qb][ks] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(d1, off + 32 * ks, qb * block_bytes, 0));
        __builtin_amdgcn_sched_barrier(0);
    };
    auto scale_owner = [&]() {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int ks = 0; ks < C::KS; ++ks) xa[qb][ks] = scale_bf16x8(xa[qb][ks], c1);
        __builtin_amdgcn_sched_barrier(0);
    };
    load_owner(h, m0);                                        // scaled by c1 once the streamed tiles are requested

    f32x16 acc0[QB][MB];                           // FWD: O^T;  DQ: dQ^T;  DKDV: dK^T
    f32x16 acc1[MODE == DKDV ? QB : 1][MODE == DKDV ? MB : 1];   // DKDV: dV^T
    // Bias gradient db = sum of dS over all valid pairs: one more (small) MFMA per 16 streamed rows with an
    // all-ones A operand sums the bf16 values that also feed dQ.  v_mfma_f32_16x16x32_bf16 reads the B operand
    // of the 32-wide shape as 16 columns x 32 contraction slots: column j of its result is the sum over the
    // lanes congruent to j modulo 16 -- which owner rows and streamed rows get mixed does not matter for a
    // total -- and every row of the result holds the same 16 sums.
    f32x4 accdb[WITH_DB ? QB : 1];
    bf16x8 ones;
    if (WITH_DB) {
#pragma unroll
        for (int i = 0; i < 8; ++i) ones[i] = (bf16_t)1.0f;
    }

    // ---- streamed tile movement: HBM -> registers -> LDS ring slot
    const int ntiles = (ns + BN - 1) / BN;
    u32x4 st1[C::PER], st2[C::PER];
    // Thread tid moves chunk tid % CH of rows tid / CH + it * RPI, it = 0 .. PER - 1: one lane constant,
    // everything else is uniform (scalar registers) or a compile-time offset.
    constexpr int RPI = C::THREADS / C::CH;        // rows per pass of the workgroup over a tile
    static_assert(C::THREADS % C::CH == 0 && (C::PER == 1 || RPI % 16 == 0), "a pass must keep the LDS row shift");
    const int r0 = tid / C::CH, col0 = (tid % C::CH) * 8;
    // A tile is read through a buffer descriptor that ends with its last valid row: the hardware returns zeros
    // beyond it without touching memory.  So neither the ragged last tile nor the tiles requested past the end
    // need a clamp, a select or a branch, and nothing waits for a load before its data is stored.  (With selects
    // behind the load the last three requests of every workgroup waited for memory on the spot: forward of one
    // 1000-token sequence 21.4 -> 19.6 us, d = 128 dK/dV at N = 2048 0.354 -> 0.337 ms.)  The descriptors advance
    // tile by tile in scalar registers; the byte offset inside a tile is a lane constant, that of a pass a scalar one.
    // Both count towards the range, also where the scalar offset alone is beyond the end (a pass that holds no valid row):
    // with Inf and NaN behind every end no output bit changes.  (Clamping it cost 0.2-0.6 %.)
    const unsigned ld_off0 = ((unsigned)r0 * (unsigned)row_stride + (unsigned)col0) * 2u;
    const unsigned pass_bytes = (unsigned)RPI * (unsigned)row_stride * 2u;
    // The stream goes on from one owner tile to the next: behind the last tile of a pass over the streamed rows
    // comes the first tile of the next pass, of the next head where the owner tiles of this one are done.
    const bf16_t *head1 = y1 + seq_base_s + (size_t)h * D, *head2 = y2 + seq_base_s + (size_t)h * D;
    const bf16_t *next1 = head1, *next2 = head2;                    // first row of the tile that is requested next
    int rows_left = ns;                                             // valid rows from there on (none past the end)
    int passes_left = left, tiles_of_head = valid_tiles - m0 / C::BM;   // passes with this one; those of this head
    auto load_tile = [&]() {
        // readfirstlane: without it the compiler moved some of this uniform state to vector registers and wrapped
        // every load in a loop over the "different" descriptors of the lanes
        const int bytes = __builtin_amdgcn_readfirstlane((rows_left < BN ? rows_left : BN) * (int)row_stride * 2);
        const auto d1 = __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(next1), 0, bytes, 0x00027000);
        const auto d2 = __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(next2), 0, bytes, 0x00027000);
#pragma unroll
        for (int it = 0; it < C::PER; ++it) {
            st1[it] = __builtin_amdgcn_raw_buffer_load_b128(d1, (int)ld_off0, it * (int)pass_bytes, 0);
            st2[it] = __builtin_amdgcn_raw_buffer_load_b128(d2, (int)ld_off0, it * (int)pass_bytes, 0);
        }
        next1 += (size_t)BN * row_stride;
        next2 += (size_t)BN * row_stride;
        rows_left = rows_left > BN ? rows_left - BN : 0;
        // d = 64: a branch that is rarely taken (N = 8192, forward + backward: 1533 us; with selects 1557).  d = 128:
        // selects, since the forward pass comes here inside a tile (12 x 1537 rows, H = 16: 162 us; with the branch 165).
        if constexpr (D == 64) {
            if (rows_left == 0 && passes_left > 1) {
                --passes_left;
                if (--tiles_of_head == 0) {
                    tiles_of_head = valid_tiles;
                    head1 += D;
                    head2 += D;
                }
                next1 = head1;
                next2 = head2;
                rows_left = ns;
            }
        } else {
            const int wrap = (rows_left == 0) & (passes_left > 1);
            passes_left -= wrap;
            tiles_of_head -= wrap;
            const int turn = wrap & (tiles_of_head == 0);
            tiles_of_head = turn ? valid_tiles : tiles_of_head;
            head1 += turn ? D : 0;
            head2 += turn ? D : 0;
            next1 = wrap ? head1 : next1;
            next2 = wrap ? head2 : next2;
            rows_left = wrap ? ns : rows_left;
        }
    };
    bf16_t *const w1 = y1s + r0 * LD1 + lds_shift<C::LM1>(r0) + col0;   // LDS home of this thread's chunk, pass 0, slot 0
    bf16_t *const w2 = y2s + r0 * LD2 + lds_shift<C::LM2>(r0) + col0;
    auto store_tile = [&](int slot) {
#pragma unroll
        for (int it = 0; it < C::PER; ++it) {
            *reinterpret_cast<u32x4 *>(w1 + (slot * BN + it * RPI) * LD1) = st1[it];
            *reinterpret_cast<u32x4 *>(w2 + (slot * BN + it * RPI) * LD2) = st2[it];
        }
    };

    // lane-constant pieces of the LDS addresses
    const int i16 = lane & 15, g16 = (lane >> 4) & 1;
    using TL1 = TrLayout<C::LM1>;
    using TL2 = TrLayout<C::LM2>;
    const int tr_row = 4 * g + (i16 >> 2);         // transposed A operand: rows 4 g + 0..3 (and + 8)
    // 16 output rows (head-dim columns) per 16-lane group; block and tile offsets are multiples of 16 rows and
    // leave the shift of a row unchanged, so every address stays a lane constant plus an immediate
    const bf16_t *rd1 = y1s + c * LD1 + lds_shift<C::LM1>(c) + 8 * g;     // row-wise A operand: row c, columns 16 ks + 8 g
    const bf16_t *rd2 = y2s + c * LD2 + lds_shift<C::LM2>(c) + 8 * g;
    const bf16_t *tr1 = y1s + tr_row * LD1 + lds_shift<C::LM1>(tr_row) + TL1::GROUP_COLS * g16 + 4 * (i16 & 3);
    const bf16_t *tr2 = y2s + tr_row * LD2 + lds_shift<C::LM2>(tr_row) + TL2::GROUP_COLS * g16 + 4 * (i16 & 3);

    // Score accumulators and bf16 operands, double buffered by block parity.
    f32x16 sbuf[2][QB], dbuf[2][Q2];
    u32x4 pbuf[2][QB][2], dsbuf[2][Q2][2];
    bf16x8 ring[RING];

    // The J-th A operand counted from the start of the step on block nb of `slot` (J >= NOPS runs into the
    // following step): row-wise operands belong to the block after the step's block, transposed ones to the
    // block before it.
    auto fetch = [&](auto J_, auto slot, auto nb_c) -> bf16x8 {
        constexpr int J = decltype(J_)::value;
        constexpr int sstep = J / NOPS, j = J % NOPS;
        constexpr int blk = decltype(nb_c)::value + sstep + (j < NA ? 1 : -1) + NB;   // >= 0, counted from the previous tile
        constexpr int tile = blk / NB - 1;                                            // relative to the current one
        constexpr int brow = (blk % NB) * 32;
        const int row = ((slot.get() + tile) & (C::NBUF - 1)) * BN + brow;
        if constexpr (j < NA) {
            constexpr int ks = j / NT, which = j % NT;
            if constexpr (which == 0) return lds_read_rows(rd1 + row * LD1 + 16 * ks);
            else return lds_read_rows(rd2 + row * LD2 + 16 * ks);
        } else {
            constexpr int jj = j - NA, which = jj % NO, idx = jj / NO, half = idx / MB, mb = idx % MB;
            // FWD contracts V^T (tensor 2); DQ contracts K^T (tensor 1); DKDV: Q^T (1) for dK, dO^T (2) for dV
            constexpr bool second = (MODE == FWD) || (MODE == DKDV && which == 1);
            if constexpr (second) {
                const bf16_t *a = tr2 + (row + 16 * half) * LD2 + TL2::MB_COLS * mb;
                return lds_read_tr(a, a + 8 * LD2 + TL2::HI_EXTRA);
            } else {
                const bf16_t *a = tr1 + (row + 16 * half) * LD1 + TL1::MB_COLS * mb;
                return lds_read_tr(a, a + 8 * LD1 + TL1::HI_EXTRA);
            }
        }
    };

    // VALU work of one step: see ValuOrder.  Per unit u (registers 2w, 2w + 1 of owner block qb = u / 8):
    //   0,1  e = 2^t'            2,3  y = 1 + cb e          4,5  P = 1 / y
    //   FWD : pack P
    //   bwd : g = e P (2 ops), a = P dP (2 ops), dS / cb = g a (2 ops), pack it, DKDV also packs P
    // 1 - P = cb e P holds without cancellation however close P is to 1, so dS = P (1 - P) dP keeps its
    // relative accuracy on the saturated tail; the constant cb is applied once, to the finished sums.
    // e = +inf (score far below the bias) meets P = 0 there: the product must be 0, not NaN.
    // Streamed rows beyond the valid length are zeros in LDS; their P and dS are set to 0 once per owner tile (mask_block).
    constexpr int OPU = (MODE == FWD) ? 7 : (MODE == DQ ? 13 : 14);

    // One pipeline step on the block (slot, nb) of parity PAR (compile-time nb).  Slots run in program
    // order; a scheduling fence closes each of them.
    // When the next tile is requested: behind the barrier that ends a tile, or right behind the stores of the one before
    // (a quarter of a tile earlier), which only the d = 128 forward pass gains from (12 x 1537 rows, H = 16: 172 -> 167 us;
    // d = 64, N = 8192, forward + backward 1543 -> 1559 us).
    constexpr bool LOAD_EARLY = MODE == FWD && D == 128;
    auto step = [&](auto has_prev_c, auto has_next_c, auto drain_c, auto nb_c, auto slot, auto store_at_c, const int store_slot) {
        constexpr int STORE_AT = decltype(store_at_c)::value;   // slot before which the staged tile goes to LDS (-1: never)
        constexpr bool HAS_PREV = decltype(has_prev_c)::value;  // a block went before: its output contractions
        constexpr bool HAS_NEXT = decltype(has_next_c)::value;  // a block follows: compute its scores
        constexpr bool DRAIN = decltype(drain_c)::value;        // only the output contractions of the last block
        constexpr int nb = decltype(nb_c)::value;
        constexpr int PAR = nb & 1;
        constexpr int G0 = (nb * NOPS) % RING;               // ring position of this step's first operand
        constexpr ValuOrder<C::UNITS, OPU, 2, 6> order{};
        constexpr int LEN = DRAIN ? 0 : C::UNITS * OPU;
        const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        float pv[HAS2 ? C::UNITS : 1][2];          // y, then P, of the units in flight (backward only)

        static_for<0, SLOTS>([&](auto k_) {
            constexpr int k = decltype(k_)::value;
            constexpr int j = k / QB, qb = k % QB;
            // The two waves of a SIMD compete for its issue port, and the older one always wins: it reached the tile
            // barrier early and left the other to finish alone, at the poor rate of a lone wave.  Priorities that
            // fall with every quarter of a tile let the wave that is behind catch up: as fast as no barrier at all
            // (N = 8192, d = 64: dK/dV 0.766 -> 0.747 ms, dQ 0.629 -> 0.611 ms; without the barrier 0.746, 0.613).
            if constexpr (!DRAIN) {
                constexpr int QUARTER = (2 * nb + (k >= SLOTS / 2)) * 4 / (2 * NB);
                if constexpr (k == 0 || k == SLOTS / 2) __builtin_amdgcn_s_setprio(3 - QUARTER);
            }
            if constexpr (k == STORE_AT) {
                store_tile(store_slot);
                if constexpr (LOAD_EARLY) load_tile();
                __builtin_amdgcn_sched_barrier(0);
            }
            // ---- the MFMA of this slot
            if constexpr (j < NA) {
                if constexpr (HAS_NEXT && !DRAIN) {
                    constexpr int ks = j / NT, which = j % NT;
                    if constexpr (which == 0)
                        sbuf[PAR ^ 1][qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            ring[(G0 + j) % RING], xa[qb][ks], ks == 0 ? zero : sbuf[PAR ^ 1][qb], 0, 0, 0);
                    else
                        dbuf[PAR ^ 1][HAS2 ? qb : 0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            ring[(G0 + j) % RING], xb[HAS2 ? qb : 0][HAS2 ? ks : 0],
                            ks == 0 ? zero : dbuf[PAR ^ 1][HAS2 ? qb : 0], 0, 0, 0);
                }
            } else if constexpr (HAS_PREV) {
                constexpr int jj = j - NA, which = jj % NO, idx = jj / NO, half = idx / MB, mb = idx % MB;
                const bf16x8 a = ring[(G0 + j) % RING];
                if constexpr (MODE == FWD) {            // O^T += V^T P^T
                    acc0[qb][mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        a, __builtin_bit_cast(bf16x8, pbuf[PAR ^ 1][qb][half]), acc0[qb][mb], 0, 0, 0);
                } else if constexpr (which == 0) {      // dQ^T += K^T dS^T   |   dK^T += Q^T dS
                    acc0[qb][mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        a, __builtin_bit_cast(bf16x8, dsbuf[PAR ^ 1][HAS2 ? qb : 0][half]), acc0[qb][mb], 0, 0, 0);
                    if constexpr (WITH_DB && mb == MB - 1)
                        accdb[qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            ones, __builtin_bit_cast(bf16x8, dsbuf[PAR ^ 1][HAS2 ? qb : 0][half]), accdb[qb], 0, 0, 0);
                } else {                                // dV^T += dO^T P
                    acc1[MODE == DKDV ? qb : 0][MODE == DKDV ? mb : 0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        a, __builtin_bit_cast(bf16x8, pbuf[PAR ^ 1][qb][half]),
                        acc1[MODE == DKDV ? qb : 0][MODE == DKDV ? mb : 0], 0, 0, 0);
                }
            }
            // ---- the register of the previous operand is free now: request the operand RING - 1 ahead
            constexpr int ahead = j + RING - 1;         // those of contractions that are not made are not read
            constexpr bool wanted = ahead < NA ? HAS_NEXT : (ahead < NOPS ? HAS_PREV : !DRAIN && (HAS_NEXT || ahead >= NOPS + NA));
            if constexpr (qb == 0 && wanted) {
                ring[(G0 + j + RING - 1) % RING] = fetch(IntC<j + RING - 1>{}, slot, nb_c);
            }
            // ---- this slot's share of the sigmoid
            static_for<(k * LEN) / SLOTS, ((k + 1) * LEN) / SLOTS>([&](auto i_) {
                constexpr int i = decltype(i_)::value;
                constexpr int u = order.unit[i], o = order.op[i];
                constexpr int uq = u / 8, w = u % 8, ra = 2 * w, rb = 2 * w + 1;
                f32x16 &s = sbuf[PAR][uq];
                f32x16 &dp = dbuf[PAR][HAS2 ? uq : 0];
                // the forward pass turns the score register into y and P in place; the backward passes keep
                // e = 2^t' there and carry y, then P, in pv
                constexpr int pu = HAS2 ? u : 0;
                auto y_of = [&](auto which) -> float {
                    if constexpr (HAS2) return pv[pu][decltype(which)::value];
                    else return s[decltype(which)::value ? rb : ra];
                };
                auto set_y = [&](auto which, const float val) {
                    if constexpr (HAS2) pv[pu][decltype(which)::value] = val;
                    else s[decltype(which)::value ? rb : ra] = val;
                };
                constexpr IntC<0> A_{};
                constexpr IntC<1> B_{};
                if constexpr (o == 0) s[ra] = __builtin_amdgcn_exp2f(s[ra]);
                else if constexpr (o == 1) s[rb] = __builtin_amdgcn_exp2f(s[rb]);
                else if constexpr (o == 2) set_y(A_, __builtin_fmaf(cb, s[ra], 1.0f));
                else if constexpr (o == 3) set_y(B_, __builtin_fmaf(cb, s[rb], 1.0f));
                else if constexpr (o == 4) set_y(A_, __builtin_amdgcn_rcpf(y_of(A_)));
                else if constexpr (o == 5) set_y(B_, __builtin_amdgcn_rcpf(y_of(B_)));
                else {
                    constexpr int e = o - 6;          // position in the mode's tail of the unit
                    if constexpr (MODE == FWD) {
                        pbuf[PAR][uq][w / 4][w % 4] = pack_bf16(s[ra], s[rb]);
                    } else {
                        if constexpr (e == 0) s[ra] = mul_zero_wins(s[ra], y_of(A_));
                        else if constexpr (e == 1) s[rb] = mul_zero_wins(s[rb], y_of(B_));
                        else if constexpr (e == 2) dp[ra] = y_of(A_) * dp[ra];
                        else if constexpr (e == 3) dp[rb] = y_of(B_) * dp[rb];
                        else if constexpr (e == 4) dp[ra] = s[ra] * dp[ra];
                        else if constexpr (e == 5) dp[rb] = s[rb] * dp[rb];
                        else if constexpr (e == 6) dsbuf[PAR][HAS2 ? uq : 0][w / 4][w % 4] = pack_bf16(dp[ra], dp[rb]);
                        else pbuf[PAR][uq][w / 4][w % 4] = pack_bf16(y_of(A_), y_of(B_));
                    }
                }
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    using T_ = IntC<1>;
    using F_ = IntC<0>;

    // ---- prologue: tiles 0 and 1 of the stream into the ring, tile 2 into registers
    {   // the first three tiles are requested back to back, so their latencies overlap
        load_tile();
        u32x4 a1[C::PER], a2[C::PER];
#pragma unroll
        for (int it = 0; it < C::PER; ++it) { a1[it] = st1[it]; a2[it] = st2[it]; }
        load_tile();
        u32x4 b1[C::PER], b2[C::PER];
#pragma unroll
        for (int it = 0; it < C::PER; ++it) { b1[it] = st1[it]; b2[it] = st2[it]; }
        load_tile();
        scale_owner();                             // the owner rows, requested first, arrive first
#pragma unroll
        for (int it = 0; it < C::PER; ++it) {
            *reinterpret_cast<u32x4 *>(w1 + (it * RPI) * LD1) = a1[it];
            *reinterpret_cast<u32x4 *>(w2 + (it * RPI) * LD2) = a2[it];
            *reinterpret_cast<u32x4 *>(w1 + (BN + it * RPI) * LD1) = b1[it];
            *reinterpret_cast<u32x4 *>(w2 + (BN + it * RPI) * LD2) = b2[it];
        }
    }

    // ---- the steps of an owner tile: block 0, which has no block before it; all blocks up to the last tile's first
    // one; the last tile's other blocks, the last of which has no successor; a step that only drains.  The loop is
    // unrolled over the four ring slots so that every LDS address is a lane constant plus an immediate.
    // Tile t + 2 goes to slot (t + 2) % 4 = (t - 2) % 4, last read during the first step of tile t - 1 (as
    // the previous block); every wave passed the barrier that ended tile t - 1.  The staged registers are
    // written half-way through the last step of tile t, and the barrier that ends the tile waits only until
    // those writes have left the LDS queue: LDS operations of a wave complete in order, so it is enough to
    // let the READS_AFTER operand reads issued behind them stay in flight.  The tile becomes visible at
    // that barrier, most of a tile before its first read near the end of tile t + 1.
    // Here t counts through all owner tiles of the workgroup: at the last tile of one the first ones of the next are
    // on their way (past the end zeros, which are not stored), so that the next one starts without waiting for memory.
    constexpr auto reads_from = [](int first_slot) {
        int cnt = 0;
        for (int k = first_slot; k < SLOTS; k += QB) {
            const int j = (k / QB + RING - 1) % NOPS;
            cnt += (j < NA) ? 1 : 2;           // one 16-byte read, or two transposing 8-byte reads
        }
        return cnt;
    };
    constexpr int STORE_AT = [&] {             // about half-way, later if too many reads would follow
        int k = (SLOTS / 2 / QB) * QB;
        while (reads_from(k) > 12) k += QB;
        return k;
    }();
    constexpr int READS_AFTER = reads_from(STORE_AT);
    static_assert(READS_AFTER <= 15 && STORE_AT < SLOTS, "more reads behind the tile store than the LDS counter can express");
    using StoreAt = IntC<STORE_AT>;
    using NoStore = IntC<-1>;
    auto tile_body = [&](auto slot_c) {            // from the second block of a tile through the first of the next
        constexpr int slot = decltype(slot_c)::value;
        static_for<1, NB>([&](auto nb_) {
            if constexpr (decltype(nb_)::value + 1 < NB) step(T_{}, T_{}, F_{}, nb_, slot_c, NoStore{}, 0);
            else step(T_{}, T_{}, F_{}, nb_, slot_c, StoreAt{}, (slot + 2) & (C::NBUF - 1));
        });
        asm volatile("s_waitcnt lgkmcnt(%0)\n\ts_barrier" ::"n"(READS_AFTER) : "memory");
        if constexpr (!LOAD_EARLY) load_tile();
        step(T_{}, T_{}, F_{}, IntC<0>{}, IntC<(slot + 1) & (C::NBUF - 1)>{}, NoStore{}, 0);
    };
    // P and dS of the streamed rows behind the valid length, in block nb of the last tile: exact zeros, as packed for the
    // output contractions.  Against a finite owner row they would add zeros anyway (the rows are zeros in LDS), but an Inf
    // in the owner row makes their scores 0 x Inf = NaN.  Two instructions a mask and one or two to apply it, on eight
    // packed pairs a block, once per owner tile and none of them in the loop.  A block without such rows is passed over,
    // but not the first one of dK/dV: with that branch the four-wave kernel reloaded four spilled registers in every tile.
    const int tail = ns - (ntiles - 1) * BN;       // valid rows of the last tile
    auto mask_block = [&](auto nb_c) {
        constexpr int nb = decltype(nb_c)::value, PAR = nb & 1;
        if ((nb > 0 || MODE != DKDV) && tail >= 32 * (nb + 1)) return;           // uniform
        const short valid = (short)(tail - 32 * nb - 4 * (fresh_lane() >> 5));   // rows of this lane, counted as below
        const s16x2 limit = {valid, valid};
#pragma unroll
        for (int w = 0; w < 8; ++w) {              // pair w holds rows 8 (w / 2) + 2 (w % 2) and the one behind it (+ 4 g)
            const short row = (short)(8 * (w / 2) + 2 * (w % 2));
            const s16x2 rows = {row, (short)(row + 1)};
            const unsigned keep = __builtin_bit_cast(unsigned, (s16x2)((rows - limit) >> 15));
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                if (MODE != DQ) pbuf[PAR][qb][w / 4][w % 4] &= keep;
                if (HAS2) dsbuf[PAR][HAS2 ? qb : 0][w / 4][w % 4] &= keep;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    int slot_rt = 0;                               // ring slot of the tile in hand
    for (;;) {
        // the tiles stored last are visible, and nobody reads the slot that is written next
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    acc0[qb][mb][i] = 0.f;
                    if (MODE == DKDV) acc1[MODE == DKDV ? qb : 0][MODE == DKDV ? mb : 0][i] = 0.f;
                }
            if (WITH_DB)
#pragma unroll
                for (int i = 0; i < 4; ++i) accdb[WITH_DB ? qb : 0][i] = 0.f;
        }
        {
            const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < C::KS; ++ks) {
                const bf16x8 a1 = lds_read_rows(rd1 + slot_rt * BN * LD1 + 16 * ks);
#pragma unroll
                for (int qb = 0; qb < QB; ++qb)
                    sbuf[0][qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, xa[qb][ks], ks == 0 ? zero : sbuf[0][qb], 0, 0, 0);
                if (HAS2) {
                    const bf16x8 a2 = lds_read_rows(rd2 + slot_rt * BN * LD2 + 16 * ks);
#pragma unroll
                    for (int qb = 0; qb < QB; ++qb)
                        dbuf[0][qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a2, xb[qb][ks], ks == 0 ? zero : dbuf[0][qb], 0, 0, 0);
                }
            }
        }
        // operands 0 .. RING - 2 of the first step
        static_for<0, RING - 1>([&](auto J_) {
            if constexpr (decltype(J_)::value < NA) ring[decltype(J_)::value % RING] = fetch(J_, DynInt{slot_rt}, IntC<0>{});
        });
        step(F_{}, T_{}, F_{}, IntC<0>{}, DynInt{slot_rt}, NoStore{}, 0);

        int t = ntiles - 1;
        while (t > 0) {
            if (slot_rt == 0) { tile_body(IntC<0>{}); slot_rt = 1; --t; }
            if (t > 0 && slot_rt == 1) { tile_body(IntC<1>{}); slot_rt = 2; --t; }
            if (t > 0 && slot_rt == 2) { tile_body(IntC<2>{}); slot_rt = 3; --t; }
            if (t > 0 && slot_rt == 3) { tile_body(IntC<3>{}); slot_rt = 0; --t; }
        }

        // ---- last tile.  The owner rows are not needed any more: request those of the next owner tile.
        const int h_done = h, m0_done = m0;
        const bool more = left > 1;
        m0 += C::BM;
        if (m0 >= n) { m0 = 0; ++h; }
        if (more) load_owner(h, m0);
        {
            const DynInt slot{slot_rt};
            mask_block(IntC<0>{});
            static_for<1, NB>([&](auto nb_) {
                step(T_{}, IntC<(decltype(nb_)::value + 1 < NB) ? 1 : 0>{}, F_{}, nb_, slot, NoStore{}, 0);
                mask_block(nb_);
            });
            const DynInt slot_next{(slot_rt + 1) & (C::NBUF - 1)};
            step(T_{}, F_{}, T_{}, IntC<0>{}, slot_next, NoStore{}, 0);
            if (more) {
                store_tile((slot_rt + 2) & (C::NBUF - 1));
                load_tile();
            }
        }

        if constexpr (WITH_DB) {
            // Row 0 of accdb (register 0 of lanes 0..15) holds 16 partial sums that together cover every dS of
            // this wave.  Owner rows beyond the valid length carry dO = 0, hence dS = 0.  Fixed-order sums: lanes
            // by butterfly, waves through LDS, workgroups in a second kernel.
            float v = 0.f;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) v += accdb[qb][0];
            v = (lane < 16) ? v : 0.f;
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
            if (lane == 0) s_db[wave] = v;
            __syncthreads();
            if (tid == 0) {
                float t = 0.f;
#pragma unroll
                for (int w = 0; w < NW; ++w) t += s_db[w];
                p.db_part[db_slot(h_done, m0_done)] = t * cb;                // the summed values are dS / cb
            }
        }

        // ---- epilogue: transposed fp32 accumulators -> bf16 rows.  Lane (c, g) holds owner row c of each block;
        // registers 4 q4 .. 4 q4 + 3 of output block mb hold head-dim columns out_col(mb, q4) + 4 g + 0..3 of the
        // layout the transposed operand was read with (plain: 32 mb + 8 q4).  The two lanes of a row (32 apart)
        // exchange halves -- lane g = 0 takes the even q4, lane g = 1 the odd ones -- so that each lane stores
        // whole 16-byte chunks: a quarter of the store instructions and write requests of 8-byte stores.
        using TL_ACC0 = TrLayout<(MODE == FWD) ? C::LM2 : C::LM1>;      // FWD contracts V^T; DQ K^T; DKDV Q^T (acc0), dO^T (acc1)
        using TL_ACC1 = TrLayout<C::LM2>;
        const float oscale = (MODE == FWD) ? 1.0f : p.scale * cb;       // dQ and dK carry the factor `scale`; their sums are over dS / cb
        auto chunk = [&](const f32x16 &a, const int pr, const float f) {   // columns of q4 = 2 pr + g
            const unsigned e0 = pack_bf16(a[8 * pr + 0] * f, a[8 * pr + 1] * f), e1 = pack_bf16(a[8 * pr + 2] * f, a[8 * pr + 3] * f);
            const unsigned o0 = pack_bf16(a[8 * pr + 4] * f, a[8 * pr + 5] * f), o1 = pack_bf16(a[8 * pr + 6] * f, a[8 * pr + 7] * f);
            const auto s0 = __builtin_amdgcn_permlane32_swap(e0, o0, false, false);   // {lower half: e0 | o0 of g = 0, upper: of g = 1}
            const auto s1 = __builtin_amdgcn_permlane32_swap(e1, o1, false, false);
            const u32x4 w = {s0[0], s1[0], s0[1], s1[1]};
            return w;
        };
        // Stores go through descriptors that end with the padded length: rows behind it are dropped, and no branch
        // keeps the compiler from counting what is in flight when the next tile's owner rows are waited for.
        const int rows = p.N - m0_done < C::BM ? p.N - m0_done : C::BM;
        const size_t base = seq_base + (size_t)m0_done * row_stride + (size_t)h_done * D;
        const int valid_rows = n - m0_done < C::BM ? n - m0_done : C::BM;       // lanes beyond store zeros
        const int off = (int)row_offset(), valid = valid_rows * (int)row_stride * 2;
        const int bytes = __builtin_amdgcn_readfirstlane(rows * (int)row_stride * 2);
        const auto d0 = __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(p.out0 + base), 0, bytes, 0x00027000);
        const auto d1 = __builtin_amdgcn_make_buffer_rsrc(uniform_ptr((MODE == DKDV ? p.out1 : p.out0) + base), 0, bytes, 0x00027000);
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const bool ok = off + qb * block_bytes < valid;
            const u32x4 z4 = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
                for (int pr = 0; pr < 2; ++pr) {
                    const u32x4 w0 = chunk(acc0[qb][mb], pr, oscale);
                    __builtin_amdgcn_raw_buffer_store_b128(ok ? w0 : z4, d0, off + 2 * TL_ACC0::out_col(mb, 2 * pr), qb * block_bytes, 0);
                    if (MODE == DKDV) {
                        const u32x4 w1 = chunk(acc1[MODE == DKDV ? qb : 0][MODE == DKDV ? mb : 0], pr, 1.0f);
                        __builtin_amdgcn_raw_buffer_store_b128(ok ? w1 : z4, d1, off + 2 * TL_ACC1::out_col(mb, 2 * pr), qb * block_bytes, 0);
                    }
                }
            }
        }
        if (--left == 0) break;
        slot_rt = (slot_rt + 1) & (C::NBUF - 1);
        scale_owner();
    }
    zero_share();
}

template <int MODE, int D, int QB, int NW, int BN, int LD1, int LD2, int OCC, int RING, bool WITH_DB = false>
__global__ void __launch_bounds__(NW * 64, OCC) sigattn_kernel(const Params p) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ MapScratch scratch;
    __shared__ float s_db[WITH_DB ? NW : 1];                        // bias gradient: one partial per wave
    using C = Cfg<MODE, D, QB, NW, BN, LD1, LD2, RING>;
    run_pass<MODE, D, QB, NW, BN, LD1, LD2, RING, WITH_DB>(p, map_work<C::BM, C::THREADS>(p, blockIdx.x, scratch), smem, s_db);
}

// Both halves of the backward pass in one launch.  Longest sequences first: workgroups [0, first_tiles) take the dK/dV
// tiles, or with `q_first` the dQ tiles, the others those of the other pass.  Batch order: the tiles of both passes of a head follow each other, so that the
// second pass finds the head's rows in the XCD's L2.
template <int D, int NW, int BN, int LD1, int LD2, int OCC, int RING_KV, int RING_Q>
__global__ void __launch_bounds__(NW * 64, OCC) sigattn_bwd_kernel(const Params kv, const Params q, const int q_first,
                                                                        const int first_tiles) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ MapScratch scratch;
    __shared__ float s_db[1];
    using C = Cfg<DKDV, D, 1, NW, BN, LD1, LD2, RING_KV>;
    const int id = blockIdx.x;
    Work w;
    bool is_kv;
    if (kv.groups) {
        int z, lo, cnt;
        batch_order_range(id, kv.wide_seqs, kv.wide_groups + q.wide_groups, kv.groups + q.groups, z, lo, cnt);
        const int pos = batch_order_pos(id, lo, cnt, shared_turn(z, cnt));
        const int kv_groups = z < kv.wide_seqs ? kv.wide_groups : kv.groups;
        const int g_kv = pos * kv_groups / cnt;                     // dK/dV workgroups in front of this one, evenly spread
        is_kv = (pos + 1) * kv_groups / cnt > g_kv;
        w = is_kv ? batch_order_share<C::BM>(kv, z, g_kv, kv_groups)
                  : batch_order_share<C::BM>(q, z, pos - g_kv, cnt - kv_groups);
    } else if (kv.in_order) {
        const int t_kv = owner_tiles<C::BM>(kv), t_q = owner_tiles<C::BM>(q);
        int tile;
        batch_order_tile(id, kv.H, t_kv + t_q, w.z, w.h, tile);
        is_kv = tile < t_kv;
        w.n = owner_length(is_kv ? kv : q, w.z);
        w.m0 = (is_kv ? tile : tile - t_kv) * C::BM;
        w.count = 1;
        w.share = w.shares = 0;
    } else {
        is_kv = (id < first_tiles) != (q_first != 0);
        const int rest = id < first_tiles ? id : id - first_tiles;
        w = is_kv ? map_work<C::BM, C::THREADS>(kv, rest, scratch) : map_work<C::BM, C::THREADS>(q, rest, scratch);
    }
    if (is_kv) run_pass<DKDV, D, 1, NW, BN, LD1, LD2, RING_KV, false>(kv, w, smem, s_db);
    else run_pass<DQ, D, 1, NW, BN, LD1, LD2, RING_Q, false>(q, w, smem, s_db);
}

// Second stage of the bias gradient: db[z] = sum of the `per_seq` partials of sequence z, in a fixed order
// (thread t takes partials t, t + 256, ...; then a tree in LDS), so the result is bitwise reproducible.
// One workgroup per sequence.
__global__ void __launch_bounds__(256) sigattn_db_reduce(const float *part, int per_seq, float *db) {
    __shared__ float s[256];
    const int z = blockIdx.x;
    float t = 0.f;
    for (int i = threadIdx.x; i < per_seq; i += 256) t += part[(size_t)z * per_seq + i];
    s[threadIdx.x] = t;
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) db[z] = s[0];
}

}  // namespace sigattn
