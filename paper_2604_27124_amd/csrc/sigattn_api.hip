// Host side of libsigattn: argument validation, kernel selection and launch behind the C ABI
// declared in include/sigmoid_attn.h.  Validation happens before any HIP call.
#include "sigattn_kernels.hpp"
#include "sigattn_onepass.hpp"
#include "sigattn_pair.hpp"
#include "sigmoid_attn.h"

#include <cmath>
#include <mutex>

using namespace sigattn;

// Scratch of the entry point that allocates nothing: one array per GPU the library runs on, held until the
// process ends.  In host code this name is only a stand-in; the array's device address comes from
// hipGetSymbolAddress, once per device (static_scratch() below), and only that pointer is ever handed on.
static __device__ __align__(256) unsigned char scratch[SIGATTN_STATIC_SCRATCH_BYTES];

namespace {

int check_shape(int B, int N, int H, int d) {
    if (B <= 0 || N <= 0 || H <= 0) return SIGATTN_ERR_INVALID_ARG;
    if (d != 64 && d != 128) return SIGATTN_ERR_UNSUPPORTED_D;
    if ((long long)B * H > 2147483647LL) return SIGATTN_ERR_TOO_LARGE;     // grid.x limit
    if ((long long)B * N * H * d >= (1LL << 40)) return SIGATTN_ERR_TOO_LARGE;
    static_assert(pair::MAX_ROW_BYTES == (1LL << 20) * (long long)sizeof(bf16_t), "longest row");
    if ((long long)H * d > (1LL << 20)) return SIGATTN_ERR_TOO_LARGE;      // 32-bit lane offsets within one streamed tile
    if (B > 256 && (long long)N > 262144LL) return SIGATTN_ERR_TOO_LARGE;  // a documented limit; the work mapping no longer needs it
    return SIGATTN_OK;
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Work mapping of a launch of `wgs` workgroups (two to a CU, 512 in flight): 1 = batch order, 0 = longest sequences
// first.  Ranking B sequences costs every workgroup about 0.08 B us of the 5 us + 0.9 us per streamed 64-row tile
// it lives (measured with the wavefronts of both workgroups ranking at once); batch order costs about half a
// workgroup's life at the end of the launch, so 0.5 / (wgs / 512) of its time.  Batch order where that is less,
// or where the ranking has no class for every tile count.  Measured, sorted against batch order, us: dK/dV + dQ
// at B = 512, N = 512: 2106 / 1850; B = 32, H = 32, N = 512: 225 / 191; B = 16, H = 32, N = 1024: 326 / 309; B = 16, H = 12,
// N = 4096 (just below the line): 951 / 946; B = 24, H = 12, N = 4096: 2179 / 2182; B = 4, H = 32, N = 4096: 953 / 972;
// B = 8, H = 12, N = 2048: 125 / 132; forward at B = 24, H = 12, N = 1500: 72 / 78.
// The host does not know the lengths.  Near the line, a batch of 64-row sequences with a long one at its end (or every
// tenth) loses by batch order what other spreads gain: forward at B = 40, H = 12, N = 1000 one 30 / 35, every tenth 37 / 42,
// uniform 90 / 87, lognormal 31 / 24, all valid 153 / 142; backward 80 / 55, 114 / 79, 299 / 274, 88 / 49, 543 / 500.
int batch_order(const Params &p, long long wgs, int owner_rows) {
    if (p.B > MAP_WAVE_B && ((long long)p.N + owner_rows - 1) / owner_rows > MAP_CLASSES) return 1;
    return p.B * wgs > 16000 + 45LL * p.N_str;
}

template <class Kern, class... Args>
int enqueue(Kern kern, long long wgs, int threads, size_t lds, hipStream_t stream, Args... args) {
    if (wgs > 2147483647LL) return SIGATTN_ERR_TOO_LARGE;
    if (lds > 65536) {   // more dynamic LDS than the default limit: opt in (idempotent, host-side only)
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds) != hipSuccess)
            return SIGATTN_ERR_LAUNCH;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)wgs, 1, 1), dim3(threads, 1, 1), lds, stream, args...);
    return hipGetLastError() == hipSuccess ? SIGATTN_OK : SIGATTN_ERR_LAUNCH;
}

template <class C>
long long tiles_of(const Params &p) {                                       // one workgroup per owner tile
    return ((long long)p.N + C::BM - 1) / C::BM * p.B * p.H;
}

// Batch order: owner tiles of a workgroup.  From the second on a tile costs no start (mapping, first loads: about 5 us of
// a workgroup's life), while the last workgroups of the launch leave CUs idle for about half their life.  With R tiles
// for each of the `slots` workgroups in flight and about 2 us per streamed 64-row tile the sum of both is least near a
// multiple of the square root of R / (streamed tiles); below R = 5 the end of the launch counts for more.  Forward +
// backward with 1 / 2 / 3 / 4 / 6 tiles, us: B = 512, H = 12, N = 512 1092 / 1061 / 1036 / 1028 / 1048; B = 200, H = 8,
// N = 100 64 / 58 / 57 / 57 / 58; B = 128, H = 12, N = 1024 857 / 840 / 828 / 841 / 839; B = 64, H = 16, N = 700, d = 128
// 815 / 763 / 755 / 774 / 768; B = 24, H = 12, N = 1500 391 / 388 / 389 / 395 / 403; B = 100, H = 4, N = 300 (R < 5) 64 / 68 /
// 73 / 78 / 96.
int tiles_per_workgroup(const Params &p, long long tiles, int slots) {
    if (tiles < 5LL * slots) return 1;
    const double j = std::sqrt(4.5 * (double)tiles / slots / ((p.N_str + 63) / 64));
    return j >= 4.0 ? 4 : (int)(j + 0.5);
}

// Deals the owner tiles of every sequence to workgroups of `chain` tiles each, a quarter of that for the last quarter
// of the sequences, so that the launch ends with short ones (B = 64, H = 16, N = 700, d = 128: 751 us; all alike 769).
// At most 16384 workgroups per sequence and pass: products of two such counts stay below 2^31.
template <class C>
void deal(Params &p, int chain) {
    const long long per_seq = ((long long)p.N + C::BM - 1) / C::BM * p.H;
    auto groups = [&](int tiles) { const long long g = (per_seq + tiles - 1) / tiles; return (int)(g > 16384 ? 16384 : g); };
    p.wide_groups = groups(chain);
    p.groups = groups((chain + 3) / 4);
    p.wide_seqs = (int)(p.B * 3LL / 4);
}
long long dealt(const Params &p) { return (long long)p.wide_seqs * p.wide_groups + (long long)(p.B - p.wide_seqs) * p.groups; }

template <int MODE, int D, int QB, int NW, int BN, int LD1, int LD2, int OCC, int RING, bool WITH_DB = false>
int launch(Params p, hipStream_t stream) {
    using C = Cfg<MODE, D, QB, NW, BN, LD1, LD2, RING>;
    const long long tiles = tiles_of<C>(p);
    long long wgs = tiles;
    p.in_order = batch_order(p, tiles, C::BM);
    if (p.in_order) {
        const int chain = tiles_per_workgroup(p, tiles, 256 * OCC);
        if (chain > 1) {
            deal<C>(p, chain);
            wgs = dealt(p);
        }
    }
    return enqueue(sigattn_kernel<MODE, D, QB, NW, BN, LD1, LD2, OCC, RING, WITH_DB>, wgs, C::THREADS, C::LDS_BYTES, stream, p);
}

// dK/dV and dQ tiles in one launch (d = 64: both passes take workgroups of the same shape).
template <int D, int NW, int BN, int LD, int OCC, int RING_KV, int RING_Q>
int launch_bwd(Params kv, Params q, hipStream_t stream) {
    using C = Cfg<DKDV, D, 1, NW, BN, LD, LD, RING_KV>;
    static_assert(C::LDS_BYTES == Cfg<DQ, D, 1, NW, BN, LD, LD, RING_Q>::LDS_BYTES, "one LDS size for both passes");
    const long long kv_tiles = tiles_of<C>(kv), q_tiles = tiles_of<C>(q), tiles = kv_tiles + q_tiles;
    long long wgs = tiles;
    kv.in_order = q.in_order = batch_order(kv, tiles, C::BM) || batch_order(q, tiles, C::BM);
    if (kv.in_order) {
        const int a = tiles_per_workgroup(kv, tiles, 256 * OCC), b = tiles_per_workgroup(q, tiles, 256 * OCC);
        const int chain = a < b ? a : b;
        if (chain > 1) {
            deal<C>(kv, chain);
            deal<C>(q, chain);
            wgs = dealt(kv) + dealt(q);
        }
    }
    // Longest first holds between the passes too: the one whose workgroups stream more rows starts.  (Cross-attention,
    // 513 queries against 3001 keys: the dQ tiles, 47 streamed tiles each, had started behind all dK/dV tiles of 9
    // and ran alone at the end; forward + backward 139 us, 111 us now.)
    const int q_first = kv.N_str < q.N_str;
    return enqueue(sigattn_bwd_kernel<D, NW, BN, LD, LD, OCC, RING_KV, RING_Q>, wgs, C::THREADS, C::LDS_BYTES,
                   stream, kv, q, q_first, (int)(q_first ? q_tiles : kv_tiles));
}

// ---- launches that leave most of the GPU idle, d = 64 (sigattn_pair.hpp)

// One workgroup of 64 rows to a CU, or other kernels: a second one on a CU takes the time that the pairs save.  Other kernels /
// pairs, us: forward at B = 2, H = 2, N = 256 (16 workgroups) 6.7 / 5.7; B = 1, H = 12, N = 1000 (192) 15.2 / 11.3; B = 1, H = 2, N = 4096
// (128) 47.8 / 33.1; B = 1, H = 12, N = 2048 (384) 26.3 / 28.1; B = 4, H = 16, N = 1024 (1024) 21.7 / 30.5.  Backward at B = 2, H = 2,
// N = 256 (32) 9.2 / 7.0, N = 700 (88) 16.5 / 11.9; B = 1, H = 2, N = 4096 (256) 70.4 / 47.9; B = 2, H = 4, 200 queries, 4000 keys (32 of 63
// steps, 504 of four) 50.5 / 35.1, but B = 1, H = 12, N = 1000 (384) 22.1 / 27.6 and B = 8, H = 4, up to 500 rows (512) 13.1 / 13.2.
constexpr long long PAIR_WGS = 256;
// What the kernels can take: a head's streamed rows under one descriptor, a ranking that has a class for every tile count.
bool pair_reach(const Params &p) {
    return (long long)p.N_str * p.H * pair::D * 2 < (1LL << 31) && (p.B <= MAP_WAVE_B || (p.N + pair::BM - 1) / pair::BM <= MAP_CLASSES);
}
long long pair_tiles(const Params &p) { return ((long long)p.N + pair::BM - 1) / pair::BM * p.B * p.H; }
long long pair_steps(const Params &p) { return ((long long)p.N_str + pair::BN - 1) / pair::BN; }                 // of one workgroup

// Both passes of a backward call: a workgroup to a CU, or where those of one pass live at most half as long as those of the other, as
// many short ones besides as fit behind each other.  (With one more than 256 of about the same length, two share a CU for all their
// life.)  A workgroup's life is its steps and a start and end of about PAIR_START of them.  Other kernels / pairs, us, all
// valid and lengths from an eighth on: 40 queries, 148 keys, 64 heads (256 workgroups) 7.6 / 6.6, 7.5 / 6.4, 72 heads (288) 8.0 / 9.3, 7.8 /
// 6.6; 64 and 128, 80 heads (240) 7.1 / 6.2, 6.9 / 6.0, 88 (264) 7.5 / 9.8, 7.4 / 7.5; 200 and 400, 24 heads (264) 11.9 / 13.4, 10.6 / 8.3.
// Short ones besides: 64 and 512, 48 heads (432, room for 240) 12.4 / 10.0, 10.4 / 8.5, 56 (504, 280) 13.4 / 13.7, 12.5 / 10.0; 100 and 1000,
// 32 heads (576, 251) 21.4 / 16.3, 15.1 / 11.5; 200 and 3000, 16 heads (816, 206) 48.4 / 32.5, 44.8 / 30.7, 32 (1632, 412) 52.0 / 60.8, 48.4 / 39.8;
// 64 and 300, 128 heads (768, 535) 13.6 / 26.6, 12.3 / 24.4.
constexpr long long PAIR_START = 6;
bool pair_fits(const Params &a, const Params &b) {
    const long long ta = pair_tiles(a), tb = pair_tiles(b), la = pair_steps(a) + PAIR_START, lb = pair_steps(b) + PAIR_START;
    const long long most = la > lb ? la : lb, least = la > lb ? lb : la;
    return ta + tb <= PAIR_WGS || (most >= 2 * least && ta * la + tb * lb <= PAIR_WGS * most);
}

// Work mapping of a small launch: more sequences than a wave ranks for itself take a histogram, 1.7 us of 5 to 7, for an order that
// matters only where workgroups follow each other on a CU and differ in length.  Sorted / batch order, us, d = 64: forward at
// B = 65, H = 1, N = 64 6.0 / 4.3, B = 256 6.5 / 4.7; backward at B = 100 6.9 / 5.5; d = 128: backward at B = 256, H = 1, N = 128 (one tile a
// head) 28.8 / 24.4; at B = 128, H = 1, N = 200 (512 workgroups, two a CU) all valid 35.0 / 32.6, from an eighth on 26.1 / 26.0, one long
// sequence at the end 18.4 / 26.6.
int small_order(const Params &p, long long wgs, int owner_rows) {
    return p.B > MAP_WAVE_B && (wgs <= 256 || (p.N <= owner_rows && p.N_str <= owner_rows));
}

template <int MODE>
int launch_pair(Params p, hipStream_t stream) {
    p.in_order = small_order(p, pair_tiles(p), pair::BM);
    return enqueue(pair::sigattn_pair<MODE>, pair_tiles(p), pair::THREADS, pair::lds_bytes(MODE), stream, p);
}

int launch_pair_bwd(Params kv, Params q, hipStream_t stream) {
    kv.in_order = q.in_order = small_order(kv, pair_tiles(kv) + pair_tiles(q), pair::BM);
    const int q_first = kv.N_str < q.N_str;             // the pass whose workgroups stream more rows starts
    return enqueue(pair::sigattn_pair_bwd, pair_tiles(kv) + pair_tiles(q), pair::THREADS, pair::lds_bytes(DKDV), stream, kv, q, q_first,
                   (int)(q_first ? pair_tiles(q) : pair_tiles(kv)));
}

// ---- the same for d = 128: half the rows to a workgroup

// A workgroup to a CU (two rounds of them for both backward passes, whose other form is two launches).  Eight waves and 256
// rows / four and 128, us: forward at B = 2, H = 16, N = 1000 (256 workgroups of 128 rows) 28.2 / 23.5; N = 2048 (512) 63.2 / 80.3; B = 1,
// H = 16, N = 4096 (512) 117 / 148.  Backward at B = 1, H = 16, N = 1024 (256 of both passes) 72.5 / 36.3; B = 2, H = 16, N = 1000 (512) 76.9 /
// 66.1, with two launches 69.3; B = 4, H = 16, N = 512 (512) 48.2 / 41.9, 44.3; B = 8, H = 16, N = 512 (1024) 78.5 / 85.5.
constexpr long long HALF_WGS = 256, HALF_BWD_WGS = 512;

long long half_tiles(const Params &p) { return ((long long)p.N + 32 * half128::NW - 1) / (32 * half128::NW) * p.B * p.H; }
bool half_ranks(const Params &p) { return p.B <= MAP_WAVE_B || (p.N + 32 * half128::NW - 1) / (32 * half128::NW) <= MAP_CLASSES; }
bool half_fits(const Params &p) { return half_tiles(p) <= HALF_WGS && half_ranks(p); }

template <int MODE, int LD1, int LD2, int OCC>
int launch_half(Params p, hipStream_t stream) {
    using C = Cfg<MODE, 128, 1, half128::NW, 64, LD1, LD2, 4>;
    static_assert(C::BM == 32 * half128::NW, "tile height");
    p.in_order = small_order(p, half_tiles(p), C::BM);
    return enqueue(half128::sigattn_half<MODE, LD1, LD2, OCC>, half_tiles(p), C::THREADS, C::LDS_BYTES, stream, p);
}

int launch_half_bwd(Params kv, Params q, hipStream_t stream) {
    constexpr size_t lds_kv = Cfg<DKDV, 128, 1, half128::NW, 64, 144, 144, 4>::LDS_BYTES, lds_q = Cfg<DQ, 128, 1, half128::NW, 64, 144, 136, 4>::LDS_BYTES;
    kv.in_order = q.in_order = small_order(kv, half_tiles(kv) + half_tiles(q), 32 * half128::NW);
    const int q_first = kv.N_str < q.N_str;             // the pass whose workgroups stream more rows starts
    return enqueue(half128::sigattn_half_bwd, half_tiles(kv) + half_tiles(q), half128::NW * 64, lds_kv > lds_q ? lds_kv : lds_q, stream, kv, q,
                   q_first, (int)(q_first ? half_tiles(q) : half_tiles(kv)));
}

// ---- the backward pass of d = 64 in one launch over the scores (sigattn_onepass.hpp)

constexpr size_t ONEPASS_LIMIT = (size_t)1 << 29;      // scratch of one launch; a larger batch goes through it in slices

size_t onepass_bytes(int B, int N, int H) {            // sums of dQ in fp32, whole tiles; plan and counts of the workgroups
    const size_t heads = (size_t)B * H, tiles = ((size_t)N + onepass::BM - 1) / onepass::BM;
    return heads * (((size_t)N + onepass::BN - 1) / onepass::BN) * onepass::TILE_BYTES +
           heads * tiles * (sizeof(onepass::TileWork) + onepass::FLAGS * sizeof(int));
}

// Sequences of one launch; 0: this shape takes two passes.  One pass does five contractions for seven, but in half as many
// workgroups of twice the keys, one to a CU, each of which follows the one before it in its head: it needs three rounds of
// them (768) and heads long enough that 256-row tiles round little; heads of two tiles, of which rounding takes most, need twelve.
// Time of two passes / one, H = 12, lengths: all valid, three quarters of N, from an eighth of N on, lognormal:
//   tiles of 256 keys       about 384               about 650               about 768               about 1536              about 3072
//   N = 384       0.97 0.95 0.81 0.72     0.92 0.88 0.90 0.96     1.01 0.95 0.94 0.96     0.90 0.89 0.88 0.96     0.98 0.92 0.94 0.89
//   N = 449       1.06 0.98 0.96 0.80     1.06 0.91 1.03 0.96     1.17 0.98 1.08 0.97     1.13 0.95 0.93 0.97     1.20 0.99 1.02 1.00
//   N = 512       1.04 0.99 1.04 0.78     1.00 0.93 1.07 1.01     1.15 1.01 0.96 1.00     1.12 0.94 0.98 1.00     1.17 1.00 1.07 1.00
//   N = 576       0.97 0.88 0.86 0.65     1.12 1.15 1.10 0.99     1.13 1.19 1.07 1.08     1.03 0.98 1.09 1.14     1.11 1.15 1.07 1.03
//   N = 700       1.16 0.96 0.85 0.75     1.24 1.14 1.07 0.99     1.23 1.09 1.05 0.96     1.14 1.07 1.09 1.10     1.22 1.13 1.17 1.15
//   N = 1024      1.03 0.96 0.88 0.69     1.14 1.22 1.04 0.93     1.31 1.15 1.17 0.95     1.26 1.18 1.16 1.18     1.25 1.24 1.21 1.20
//   N = 2048      1.04 0.96 0.88 0.90     1.25 1.22 1.06 0.97     1.28 1.17 1.11 0.99     1.26 1.21 1.21 1.19     1.28 1.27 1.24 1.25
//   N = 4096      1.04 0.96 0.81 1.03     1.15 1.16 1.01 1.12     1.26 1.17 1.11 1.13     1.26 1.22 1.19 1.16     1.27 1.26 1.24 1.23
// So below 768 ragged batches lose what full ones gain, and at N <= 512 they still do at 1536 (from 3072 to 12288 tiles, 2 to 32
// heads, N = 460 and 512 0.94 to 1.29).  The host does not know the lengths:
// a batch of one long sequence among others of a sixteenth of it leaves most CUs without a tile, and one pass takes longer
// (us, two / one: B = 16, N = 1024 38 / 60; B = 8, N = 2048 67 / 114; B = 8, N = 4096 214 / 252; not from N = 8192 on, 759 / 722 at B = 4;
// H = 2, where the long one has fewest tiles: B = 85, N = 1406 33 / 87; with lognormal lengths B = 19, N = 5892 382 / 444, over 21
// such batches of two heads 0.86 to 1.28 times as fast, 1.04 on average).
int onepass_sequences(int B, int N, int H, int d) {
    const long long tiles = ((long long)N + onepass::BM - 1) / onepass::BM * H * B;
    if (d != 64 || N <= 448 || tiles < (N <= 512 ? 3072 : 768)) return 0;
    const size_t one = onepass_bytes(1, N, H);
    if (one > ONEPASS_LIMIT) return 0;
    const long long most = (long long)(ONEPASS_LIMIT / one), slices = (B + most - 1) / most;
    return (int)((B + slices - 1) / slices);           // slices of equal size
}

int launch_onepass(onepass::Params p, const int per_slice, unsigned char *workspace, hipStream_t stream) {
    const int B = p.B, T = (p.L_k + onepass::BM - 1) / onepass::BM, TQ = (p.L_q + onepass::BN - 1) / onepass::BN;
    const size_t row = (size_t)p.H * onepass::D;
    for (int z = 0; z < B; z += per_slice) {
        onepass::Params s = p;
        s.B = B - z < per_slice ? B - z : per_slice;
        const size_t q_off = (size_t)z * p.L_q * row, k_off = (size_t)z * p.L_k * row;
        s.q += q_off; s.d_o += q_off; s.dq += q_off;
        s.k += k_off; s.v += k_off; s.dk += k_off; s.dv += k_off;
        s.seqlens_q += z; s.seqlens_k += z; s.bias += z;
        s.group = onepass::plan_group(s.B, p.H, TQ);
        const long long wgs = (long long)s.B * s.H * T;
        s.part = workspace;
        s.plan = reinterpret_cast<onepass::TileWork *>(workspace + (size_t)s.B * s.H * TQ * onepass::TILE_BYTES);
        s.flags = reinterpret_cast<int *>(s.plan + wgs);
        if (int e = enqueue(onepass::sigattn_onepass_plan, (wgs + onepass::PLAN_THREADS - 1) / onepass::PLAN_THREADS, onepass::PLAN_THREADS, 0, stream, s)) return e;
        if (int e = enqueue(onepass::sigattn_onepass, wgs, onepass::THREADS, onepass::LDS_BYTES, stream, s)) return e;
    }
    return SIGATTN_OK;
}

}  // namespace

extern "C" {

int sigmoid_attn_version(void) { return 400; }

const char *sigmoid_attn_strerror(int code) {
    switch (code) {
        case SIGATTN_OK: return "success";
        case SIGATTN_ERR_INVALID_ARG: return "invalid argument (null pointer, non-positive dimension or non-finite scale)";
        case SIGATTN_ERR_UNSUPPORTED_D: return "unsupported head dimension (must be 64 or 128)";
        case SIGATTN_ERR_MISALIGNED: return "tensor pointer is not 16-byte aligned";
        case SIGATTN_ERR_WORKSPACE: return "workspace missing or too small";
        case SIGATTN_ERR_LAUNCH: return "HIP kernel launch failed";
        case SIGATTN_ERR_TOO_LARGE: return "problem too large: more workgroups than one launch holds, H*d > 2^20, more than 256 sequences padded beyond 262144 rows, or more query tiles than the static scratch array holds";
        default: return "unknown error code";
    }
}

size_t sigmoid_attn_bwd_workspace_bytes(int B, int N_max, int H, int d) {
    if (check_shape(B, N_max, H, d) != SIGATTN_OK) return 0;
    return 0;   // in two passes each workgroup owns its output tiles: no scratch, no atomics
}

size_t sigmoid_attn_bwd_onepass_workspace_bytes(int B, int N_max, int H, int d) {
    if (check_shape(B, N_max, H, d) != SIGATTN_OK) return 0;
    const int per_slice = onepass_sequences(B, N_max, H, d);
    return per_slice == 0 ? 0 : onepass_bytes(per_slice, N_max, H);
}

// ---- common implementations: separate query-side and key-side lengths (self-attention passes them twice)

static int fwd_impl(const void *q, const void *k, const void *v, void *o,
                    const int32_t *seqlens_q, const int32_t *seqlens_k, const float *bias, float scale,
                    int B, int L_q, int L_k, int H, int d, void *stream) {
    if (!q || !k || !v || !o || !seqlens_q || !seqlens_k || !bias || !std::isfinite(scale)) return SIGATTN_ERR_INVALID_ARG;
    if (int e = check_shape(B, L_q, H, d)) return e;
    if (int e = check_shape(B, L_k, H, d)) return e;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o)) return SIGATTN_ERR_MISALIGNED;

    Params p{};
    p.q = static_cast<const bf16_t *>(q);
    p.k = static_cast<const bf16_t *>(k);
    p.v = static_cast<const bf16_t *>(v);
    p.d_o = nullptr;
    p.out0 = static_cast<bf16_t *>(o);
    p.out1 = nullptr;
    p.seqlens = seqlens_q;          // owner side: queries
    p.seqlens_str = seqlens_k;      // streamed side: keys / values
    p.bias = bias;
    p.scale = scale;
    p.B = B; p.N = L_q; p.N_str = L_k; p.H = H;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (d == 64) {
        // More workgroups than CUs: four waves of two owner blocks (256 query rows, two workgroups to a CU) feed two MFMAs from every LDS
        // operand read.  A grid of at most one such workgroup per CU is split finer, into 128-row tiles (B = 4,
        // H = 16, N = 1024, 256 workgroups: 19.3 against 23.0 us; B = 8, H = 12, 384 workgroups: 32.4 against
        // 30.2 us), and sequences that fit one 128-row tile take it (B = 200, H = 8, N = 100: 19.2 against 25.1 us).
        if (pair_tiles(p) <= PAIR_WGS && pair_reach(p)) return launch_pair<FWD>(p, s);
        if (L_q <= 128 || (long long)B * H * ((L_q + 255) / 256) <= 256) return launch<FWD, 64, 1, 4, 64, 72, 72, 2, 4>(p, s);
        return launch<FWD, 64, 2, 4, 64, 72, 72, 2, 4>(p, s);
    }
    // d = 128: K is only read row-wise (272-byte rows), V only through the transposing reads, which at that
    // stride ran at a quarter of their rate; 288-byte rows with the split column layout are conflict-free.
    if (half_fits(p)) return launch_half<FWD, 136, 144, half128::OCC_FWD>(p, s);
    return launch<FWD, 128, 1, 8, 64, 136, 144, 1, 4>(p, s);
}

// Everything a backward call can be refused for; every way of making the call asks here first.
static int check_bwd(const void *q, const void *k, const void *v, const void *d_o,
                     const void *dq, const void *dk, const void *dv,
                     const int32_t *seqlens_q, const int32_t *seqlens_k, const float *bias, float scale,
                     int B, int L_q, int L_k, int H, int d, bool want_dq, bool want_dkdv) {
    if (!q || !k || !v || !d_o || !seqlens_q || !seqlens_k || !bias || !std::isfinite(scale)) return SIGATTN_ERR_INVALID_ARG;
    if ((want_dq && !dq) || (want_dkdv && (!dk || !dv))) return SIGATTN_ERR_INVALID_ARG;
    if (int e = check_shape(B, L_q, H, d)) return e;
    if (int e = check_shape(B, L_k, H, d)) return e;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(d_o)) return SIGATTN_ERR_MISALIGNED;
    if ((want_dq && !aligned16(dq)) || (want_dkdv && (!aligned16(dk) || !aligned16(dv))))
        return SIGATTN_ERR_MISALIGNED;
    return SIGATTN_OK;
}

static int bwd_impl(const void *q, const void *k, const void *v, const void *d_o,
                    void *dq, void *dk, void *dv,
                    const int32_t *seqlens_q, const int32_t *seqlens_k, const float *bias, float scale,
                    int B, int L_q, int L_k, int H, int d, void *stream, bool want_dq, bool want_dkdv) {
    if (int e = check_bwd(q, k, v, d_o, dq, dk, dv, seqlens_q, seqlens_k, bias, scale, B, L_q, L_k, H, d, want_dq, want_dkdv)) return e;

    Params p{};
    p.q = static_cast<const bf16_t *>(q);
    p.k = static_cast<const bf16_t *>(k);
    p.v = static_cast<const bf16_t *>(v);
    p.d_o = static_cast<const bf16_t *>(d_o);
    p.bias = bias;
    p.scale = scale;
    p.B = B; p.H = H;
    hipStream_t s = static_cast<hipStream_t>(stream);

    Params pk = p;           // Alg. 3: dK, dV (owner = key tile, streamed = queries and dO)
    pk.seqlens = seqlens_k; pk.N = L_k;
    pk.seqlens_str = seqlens_q; pk.N_str = L_q;
    pk.out0 = static_cast<bf16_t *>(dk);
    pk.out1 = static_cast<bf16_t *>(dv);
    Params pq = p;           // Alg. 2: dQ (owner = query tile, streamed = keys and values)
    pq.seqlens = seqlens_q; pq.N = L_q;
    pq.seqlens_str = seqlens_k; pq.N_str = L_k;
    pq.out0 = static_cast<bf16_t *>(dq);
    pq.out1 = nullptr;

    if (d == 64) {
        // Four waves (128 owner rows), two workgroups to a CU, so that one fills the other's start and end.  Eight waves
        // and 256 rows, one to a CU, halve the tile movement per owner row and still gain nothing: dK/dV + dQ with four /
        // eight, us, all rows valid: B = 1, H = 2, N = 4096 71 / 99; B = 3, H = 16, N = 3000 403 / 407, N = 8192 2704 /
        // 2683; B = 16, H = 12, N = 4096 2873 / 2828; lengths from a quarter of N on: B = 4, H = 12, N = 4096 364 / 381,
        // N = 8192 1345 / 1383; B = 1, H = 12, N = 16384 2231 / 2265.  Over 140 such cases four take 0.71 to 1.025 of the
        // time of eight.
        // One launch for both passes: one start, and the tail of the first is filled by the second (B = 2, H = 2,
        // N = 256: 9.4 us against 9.0 + 8.0; B = 12 heads of N = 1000: 22.5 against 21.9 + 19.4; N = 8192: 1.5 % less).
        if (pair_reach(pk) && pair_reach(pq)) {
            if (want_dkdv && want_dq && pair_fits(pk, pq)) return launch_pair_bwd(pk, pq, s);
            if (want_dkdv && !want_dq && pair_tiles(pk) <= PAIR_WGS) return launch_pair<DKDV>(pk, s);
            if (want_dq && !want_dkdv && pair_tiles(pq) <= PAIR_WGS) return launch_pair<DQ>(pq, s);
        }
        if (want_dkdv && want_dq) return launch_bwd<64, 4, 64, 72, 2, 8, 4>(pk, pq, s);
        if (want_dkdv) return launch<DKDV, 64, 1, 4, 64, 72, 72, 2, 8>(pk, s);
        if (want_dq) return launch<DQ, 64, 1, 4, 64, 72, 72, 2, 4>(pq, s);
        return SIGATTN_OK;
    }
    if (want_dkdv && want_dq && half_tiles(pk) + half_tiles(pq) <= HALF_BWD_WGS && half_ranks(pk) && half_ranks(pq))
        return launch_half_bwd(pk, pq, s);
    if (want_dkdv) {
        // d = 128: the fp32 accumulators of dK and dV (128 registers) fit only with the whole register file of a
        // SIMD for one wave, so four waves of 32 keys, one per SIMD (both streamed tensors are read row-wise and
        // transposed: 288-byte LDS rows).
        const int e = launch<DKDV, 128, 1, 4, 64, 144, 144, 1, 4>(pk, s);
        if (e) return e;
    }
    if (want_dq && half_fits(pq)) return launch_half<DQ, 144, 136, half128::OCC_BWD>(pq, s);
    if (want_dq) return launch<DQ, 128, 1, 8, 64, 144, 136, 1, 4>(pq, s);
    return SIGATTN_OK;
}

int sigmoid_attn_fwd(const void *q, const void *k, const void *v, void *o,
                     const int32_t *seqlens, const float *bias, float scale,
                     int B, int N_max, int H, int d, void *stream) {
    return fwd_impl(q, k, v, o, seqlens, seqlens, bias, scale, B, N_max, N_max, H, d, stream);
}

int sigmoid_attn_bwd(const void *q, const void *k, const void *v, const void *d_o,
                     void *dq, void *dk, void *dv,
                     const int32_t *seqlens, const float *bias, float scale,
                     int B, int N_max, int H, int d,
                     void *workspace, size_t workspace_bytes, void *stream) {
    // argument errors first, as the header orders them
    if (int e = check_bwd(q, k, v, d_o, dq, dk, dv, seqlens, seqlens, bias, scale, B, N_max, N_max, H, d, true, true)) return e;
    const size_t need = sigmoid_attn_bwd_workspace_bytes(B, N_max, H, d);
    if (need > 0 && (!workspace || workspace_bytes < need)) return SIGATTN_ERR_WORKSPACE;
    const size_t one = sigmoid_attn_bwd_onepass_workspace_bytes(B, N_max, H, d);
    if (one > 0 && workspace && workspace_bytes >= one && aligned16(workspace)) {
        onepass::Params p{};
        p.q = static_cast<const bf16_t *>(q);
        p.k = static_cast<const bf16_t *>(k);
        p.v = static_cast<const bf16_t *>(v);
        p.d_o = static_cast<const bf16_t *>(d_o);
        p.dq = static_cast<bf16_t *>(dq);
        p.dk = static_cast<bf16_t *>(dk);
        p.dv = static_cast<bf16_t *>(dv);
        p.seqlens_q = p.seqlens_k = seqlens;
        p.bias = bias;
        p.scale = scale;
        p.B = B; p.L_q = p.L_k = N_max; p.H = H;
        return launch_onepass(p, onepass_sequences(B, N_max, H, d), static_cast<unsigned char *>(workspace), static_cast<hipStream_t>(stream));
    }
    return bwd_impl(q, k, v, d_o, dq, dk, dv, seqlens, seqlens, bias, scale, B, N_max, N_max, H, d, stream, true, true);
}

int sigmoid_attn_bwd_dq(const void *q, const void *k, const void *v, const void *d_o, void *dq,
                        const int32_t *seqlens, const float *bias, float scale,
                        int B, int N_max, int H, int d, void *stream) {
    return bwd_impl(q, k, v, d_o, dq, nullptr, nullptr, seqlens, seqlens, bias, scale, B, N_max, N_max, H, d, stream, true, false);
}

int sigmoid_attn_bwd_dkdv(const void *q, const void *k, const void *v, const void *d_o, void *dk, void *dv,
                          const int32_t *seqlens, const float *bias, float scale,
                          int B, int N_max, int H, int d, void *stream) {
    return bwd_impl(q, k, v, d_o, nullptr, dk, dv, seqlens, seqlens, bias, scale, B, N_max, N_max, H, d, stream, false, true);
}

// Bias-gradient partials: 8 bytes per 256 query rows of every (z, h), which hold one float per tile of 128 (d = 64) or
// 256 rows (d = 128).
static long long dq_workgroups(int B, int N, int H) { return (((long long)N + 255) / 256) * B * H; }

size_t sigmoid_attn_bwd_dq_dbias_workspace_bytes(int B, int N_max, int H, int d) {
    if (check_shape(B, N_max, H, d) != SIGATTN_OK) return 0;
    return (size_t)dq_workgroups(B, N_max, H) * (sizeof(float) + sizeof(int32_t));
}

size_t sigmoid_attn_cross_bwd_dq_dbias_workspace_bytes(int B, int L_q, int L_k, int H, int d) {
    if (check_shape(B, L_k, H, d) != SIGATTN_OK) return 0;
    return sigmoid_attn_bwd_dq_dbias_workspace_bytes(B, L_q, H, d);     // sized by the query side
}

static int dq_dbias_impl(const void *q, const void *k, const void *v, const void *d_o, void *dq, float *dbias,
                         const int32_t *seqlens_q, const int32_t *seqlens_k, const float *bias, float scale,
                         int B, int L_q, int L_k, int H, int d,
                         void *workspace, size_t workspace_bytes, void *stream) {
    if (!q || !k || !v || !d_o || !dq || !dbias || !seqlens_q || !seqlens_k || !bias || !std::isfinite(scale))
        return SIGATTN_ERR_INVALID_ARG;
    if (int e = check_shape(B, L_q, H, d)) return e;
    if (int e = check_shape(B, L_k, H, d)) return e;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(d_o) || !aligned16(dq)) return SIGATTN_ERR_MISALIGNED;
    const size_t need = sigmoid_attn_bwd_dq_dbias_workspace_bytes(B, L_q, H, d);
    if (!workspace || workspace_bytes < need) return SIGATTN_ERR_WORKSPACE;
    if (!aligned16(workspace) || (reinterpret_cast<uintptr_t>(dbias) & 3u)) return SIGATTN_ERR_MISALIGNED;

    Params p{};
    p.q = static_cast<const bf16_t *>(q);
    p.k = static_cast<const bf16_t *>(k);
    p.v = static_cast<const bf16_t *>(v);
    p.d_o = static_cast<const bf16_t *>(d_o);
    p.out0 = static_cast<bf16_t *>(dq);
    p.seqlens = seqlens_q;          // owner side: queries
    p.seqlens_str = seqlens_k;      // streamed side: keys / values
    p.bias = bias;
    p.scale = scale;
    p.B = B; p.N = L_q; p.N_str = L_k; p.H = H;
    p.db_part = static_cast<float *>(workspace);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int e = (d == 64) ? launch<DQ, 64, 1, 4, 64, 72, 72, 2, 4, true>(p, s)
                            : launch<DQ, 128, 1, 8, 64, 144, 136, 1, 2, true>(p, s);
    if (e) return e;
    const int rows = (d == 64) ? 128 : 256;         // query rows of a partial sum
    hipLaunchKernelGGL(sigattn_db_reduce, dim3((unsigned)B), dim3(256), 0, s, p.db_part, (L_q + rows - 1) / rows * H, dbias);
    return hipGetLastError() == hipSuccess ? SIGATTN_OK : SIGATTN_ERR_LAUNCH;
}

int sigmoid_attn_bwd_dq_dbias(const void *q, const void *k, const void *v, const void *d_o, void *dq, float *dbias,
                              const int32_t *seqlens, const float *bias, float scale,
                              int B, int N_max, int H, int d,
                              void *workspace, size_t workspace_bytes, void *stream) {
    return dq_dbias_impl(q, k, v, d_o, dq, dbias, seqlens, seqlens, bias, scale, B, N_max, N_max, H, d,
                         workspace, workspace_bytes, stream);
}

// Device address of this GPU's copy of `scratch`: looked up on the first call on each device, with that
// device current, and kept.  Every GPU holds its own copy of the array at its own address.
static void *static_scratch() {
    constexpr int MAX_DEVICES = 64;
    static std::mutex lock;
    static void *ptr[MAX_DEVICES] = {};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return nullptr;
    std::lock_guard<std::mutex> hold(lock);
    if (!ptr[dev]) {
        void *a = nullptr;
        if (hipGetSymbolAddress(&a, HIP_SYMBOL(scratch)) != hipSuccess || !a) return nullptr;
        ptr[dev] = a;
    }
    return ptr[dev];
}

int sigmoid_attn_bwd_dq_dbias_static(const void *q, const void *k, const void *v, const void *d_o, void *dq,
                                     float *dbias, const int32_t *seqlens, const float *bias, float scale,
                                     int B, int N_max, int H, int d, void *stream) {
    // Argument errors first, on the host, exactly as the workspace form reports them (a non-null, aligned
    // stand-in of sufficient size takes the place of the workspace for that pass; nothing is launched).
    if (!q || !k || !v || !d_o || !dq || !dbias || !seqlens || !bias || !std::isfinite(scale)) return SIGATTN_ERR_INVALID_ARG;
    if (int e = check_shape(B, N_max, H, d)) return e;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(d_o) || !aligned16(dq) ||
        (reinterpret_cast<uintptr_t>(dbias) & 3u))
        return SIGATTN_ERR_MISALIGNED;
    const size_t need = sigmoid_attn_bwd_dq_dbias_workspace_bytes(B, N_max, H, d);
    if (need > (size_t)SIGATTN_STATIC_SCRATCH_BYTES) return SIGATTN_ERR_TOO_LARGE;   // more query rows than the array has room for
    void *ws = static_scratch();
    if (!ws) return SIGATTN_ERR_LAUNCH;
    // Every owner tile's partial is written and the second kernel reads exactly those: nothing has to start at zero.
    return dq_dbias_impl(q, k, v, d_o, dq, dbias, seqlens, seqlens, bias, scale, B, N_max, N_max, H, d,
                         ws, (size_t)SIGATTN_STATIC_SCRATCH_BYTES, stream);
}

int sigmoid_attn_cross_bwd_dq_dbias(const void *q, const void *k, const void *v, const void *d_o, void *dq,
                                    float *dbias, const int32_t *seqlens_q, const int32_t *seqlens_k,
                                    const float *bias, float scale, int B, int L_q, int L_k, int H, int d,
                                    void *workspace, size_t workspace_bytes, void *stream) {
    return dq_dbias_impl(q, k, v, d_o, dq, dbias, seqlens_q, seqlens_k, bias, scale, B, L_q, L_k, H, d,
                         workspace, workspace_bytes, stream);
}

int sigmoid_attn_cross_fwd(const void *q, const void *k, const void *v, void *o,
                           const int32_t *seqlens_q, const int32_t *seqlens_k, const float *bias, float scale,
                           int B, int L_q, int L_k, int H, int d, void *stream) {
    return fwd_impl(q, k, v, o, seqlens_q, seqlens_k, bias, scale, B, L_q, L_k, H, d, stream);
}

int sigmoid_attn_cross_bwd(const void *q, const void *k, const void *v, const void *d_o,
                           void *dq, void *dk, void *dv,
                           const int32_t *seqlens_q, const int32_t *seqlens_k, const float *bias, float scale,
                           int B, int L_q, int L_k, int H, int d, void *stream) {
    if (!dq || !dk || !dv) return SIGATTN_ERR_INVALID_ARG;
    return bwd_impl(q, k, v, d_o, dq, dk, dv, seqlens_q, seqlens_k, bias, scale, B, L_q, L_k, H, d, stream, true, true);
}

}  // extern "C"
