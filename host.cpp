#ifdef OLD
#include "old_schedule.cpp"
#else
#include "schedule.cpp"
#endif
#include <chrono>
#include <cstdio>
using namespace hspmd;
extern "C" double refill_us(const int* cu, int n, int hq, int hkv, int d, int reps) {
    double best = 1e18;
    for (int r = 0; r < reps; ++r) {
        auto t0 = std::chrono::steady_clock::now();
        PassLoad load[3]; for (int k = 0; k < 3; ++k) load[k] = pass_load((hspmd_list_kind)k, cu, n, hq, hkv);
        auto a = build_work_list(HSPMD_LIST_FWD, cu, n, hq, hkv, kNumXcd);
        auto b = build_work_list(HSPMD_LIST_DKV, cu, n, hq, hkv, kNumXcd);
#ifndef OLD
        PieceList p; bool dealt = build_piece_list(cu, n, hq, hkv, kNumXcd, load[2], b.size(), d, std::max(a.size(), b.size()) <= 240 ? 240 : 2147483647LL, p);
        asm volatile("" :: "r"(dealt));
#endif
        best = std::min(best, std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t0).count());
    }
    return best;
}
extern "C" double estimate_us(const int* cu, int n, int hq, int hkv, int d, int reps) {
    double best = 1e18, x = 0;
    for (int r = 0; r < reps; ++r) {
        auto t0 = std::chrono::steady_clock::now();
        for (int k = 0; k < 3; ++k) x += estimate_pass_us((hspmd_list_kind)k, cu, n, hq, hkv, d);
        best = std::min(best, std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t0).count());
    }
    return best;
}
