// The plan of a one-pass backward launch (sigattn_onepass.hpp): which key tile of which head the workgroup of an id works on.
// A kernel makes it, a thread per tile; the steps of a thread are functions of their own, so that a host program can run
// them thread by thread.
//
// A tile of keys has a larger place than the tiles before it in its head (the order of the chain), and long sequences come
// first.  A tile can only follow the one before it at a distance of about three query tiles, so tiles of one head that
// start together wait for each other; `group` sequences of neighbouring rank are therefore dealt in turn, tile by tile.  Up
// to PLAN_B sequences are ranked, by their queries (a workgroup's time); more are taken in batch order, in groups as well.
// Padded tiles, which only write zeros, come last or with their sequence.
// Time with groups of one / few / all sequences, us: 4 x 12 heads, 2958 to 7122 rows 995 / 1004 / 1034; 8 x 12 x 2048
// 325 / 303 / 299; 16 x 12 of 64 to 4096 rows 593 / 580 / 605; 4 x 12 x 8192 2345 / 2265 / 2240.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sigattn {
namespace onepass {

#define SIGATTN_BOTH __host__ __device__ __forceinline__

constexpr int BM = 256;                      // key rows of a workgroup
constexpr int BN = 64;                       // query rows of a streamed tile
constexpr int PLAN_THREADS = 256, PLAN_B = PLAN_THREADS;

// One workgroup's work: a key tile of head h of sequence z, which has nq valid queries and nk valid keys.  j counts the tiles of
// the head; of those with valid keys each workgroup takes the next one when it starts.
struct alignas(16) TileWork { int z, h, j, nq, nk; float bias; };    // as far as a workspace has to be aligned
static_assert(sizeof(TileWork) == 32, "two 16-byte accesses");

SIGATTN_BOTH int clamp_len(int v, int n) { return v < 0 ? 0 : (v > n ? n : v); }

// Sequences that are dealt in turn.  A tile of keys takes about one round of its query tiles after another, 256 at a time, and
// follows the tile before it by three of them: 768 / TQ heads in turn keep pace, four times as many leave room.
SIGATTN_BOTH int plan_group(int B, int H, int query_tiles) {
    const long long heads = (long long)H * query_tiles, turn = (3000 + heads - 1) / heads;
    return (int)(turn < B ? turn : B);
}

// What the threads of a block share: queries and rank of a sequence, tiles of a rank; tiles of the ranks before, padded tiles
// of the sequences before (each twice: a step of the prefix sums reads one and writes the other).
struct PlanScratch {
    int q[PLAN_B], rank[PLAN_B], tiles[PLAN_B];
    int before[2][PLAN_B + 1], padded[2][PLAN_B + 1];
};

// The steps of thread `tid` (B <= PLAN_B), each behind a barrier; q_len and k_len are the lengths of sequence tid.
SIGATTN_BOTH int plan_tiles(int k_len, int L_k) { return (clamp_len(k_len, L_k) + BM - 1) / BM; }
SIGATTN_BOTH void plan_take(PlanScratch &s, int tid, int B, int q_len, int L_q) { s.q[tid] = tid < B ? clamp_len(q_len, L_q) : -1; }
SIGATTN_BOTH void plan_rank(PlanScratch &s, int tid, int B, int k_len, int L_k) {
    const int q = s.q[tid];
    int rank = 0;
    for (int u = 0; u < B; ++u) rank += s.q[u] > q || (s.q[u] == q && u < tid) ? 1 : 0;
    s.rank[tid] = rank;
    if (tid < B) s.tiles[rank] = plan_tiles(k_len, L_k);
}
SIGATTN_BOTH void plan_fill(PlanScratch &s, int tid, int B, int k_len, int L_k) {
    s.before[0][tid + 1] = tid < B ? s.tiles[tid] : 0;
    s.padded[0][tid + 1] = tid < B ? (L_k + BM - 1) / BM - plan_tiles(k_len, L_k) : 0;
    if (tid == 0) s.before[0][0] = s.before[1][0] = s.padded[0][0] = s.padded[1][0] = 0;
}
constexpr int PLAN_SCANS = 8;                // steps of the inclusive prefix sums; the last one writes half 0
static_assert(1 << PLAN_SCANS == PLAN_B && PLAN_SCANS % 2 == 0, "prefix sums");
SIGATTN_BOTH void plan_scan(PlanScratch &s, int tid, int step) {
    const int off = 1 << step, from = step & 1;
    s.before[from ^ 1][tid + 1] = s.before[from][tid + 1] + (tid >= off ? s.before[from][tid + 1 - off] : 0);
    s.padded[from ^ 1][tid + 1] = s.padded[from][tid + 1] + (tid >= off ? s.padded[from][tid + 1 - off] : 0);
}

// The id of tile j of head h of sequence z, T tiles to a head.
SIGATTN_BOTH int plan_id(const PlanScratch &s, int z, int h, int j, int B, int H, int T, int group) {
    if (B > PLAN_B) {                                                // batch order
        const int z0 = z - z % group, members = B - z0 < group ? B - z0 : group;
        return z0 * H * T + (j * members + z - z0) * H + h;
    }
    const int rank = s.rank[z], mine = s.tiles[rank], lo = rank - rank % group;
    int at;                                                          // tiles of one head each in front of this one
    if (j < mine) {
        at = s.before[0][lo];
        for (int r = lo; r < lo + group && r < B; ++r) {
            const int t = s.tiles[r];
            at += (t < j ? t : j) + (r < rank && t > j ? 1 : 0);
        }
    } else {
        at = s.before[0][B] + s.padded[0][z] + j - mine;
    }
    return at * H + h;
}

}  // namespace onepass
}  // namespace sigattn
