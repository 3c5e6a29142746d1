// The plan kernel's steps, run on the CPU thread by thread: ids of all tiles, [B][H][key tiles].
#include "sigattn_onepass_plan.hpp"

#include <cstring>

using namespace sigattn::onepass;

extern "C" int plan_ids(const int *nq, const int *nk, int B, int H, int L_q, int L_k, int group, int *ids) {
    static PlanScratch s;
    memset(&s, 0x5a, sizeof s);              // LDS holds anything when the kernel starts
    const int T = (L_k + BM - 1) / BM;
    if (B <= PLAN_B) {
        auto every = [&](auto step) { for (int t = 0; t < PLAN_THREADS; ++t) step(t, t < B ? nq[t] : 0, t < B ? nk[t] : 0); };
        every([&](int t, int q, int) { plan_take(s, t, B, q, L_q); });
        every([&](int t, int, int k) { plan_rank(s, t, B, k, L_k); });
        every([&](int t, int, int k) { plan_fill(s, t, B, k, L_k); });
        for (int step = 0; step < PLAN_SCANS; ++step) every([&](int t, int, int) { plan_scan(s, t, step); });
    }
    for (int i = 0; i < B * H * T; ++i) ids[i] = plan_id(s, i / T / H, i / T % H, i % T, B, H, T, group);
    return T;
}
extern "C" int group_of(int B, int H, int query_tiles) { return plan_group(B, H, query_tiles); }
