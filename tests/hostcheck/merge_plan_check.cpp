// Random chunk plans, well formed and not: the launches of merge_chunks must
// count every (head, block) as often as running the chunks one by one does,
// write a head before folding into it, and leave exactly the uncovered heads to
// be cleared; a plan whose ranges overlap must be refused.
#include <cstdio>
#include <random>

#include "../../paper_2609_32197_amd/csrc/sparsp_launch.h"

int main() {
    std::mt19937 rng(7);
    auto in = [&](int lo, int hi) { return lo + int(rng() % unsigned(hi - lo + 1)); };
    int failures = 0, merged = 0, refused = 0, single = 0;
    for (int it = 0; it < 20000; ++it) {
        const int H = in(1, 9), n = in(1, 40);
        std::vector<sparsp_chunk> plan;
        if (it % 4 == 0) {  // a schedule of plan_chunks
            const int W = (n + 63) / 64, R = in(1, n), rank = in(0, R - 1);
            sparsp::Geom g{H, n * 4, 4, 4, 0, 1, n, 1, W, false};
            std::vector<uint64_t> demand(size_t(H) * W);
            for (auto& w : demand) w = (uint64_t(rng()) << 32 | rng()) & ((n < 64 ? uint64_t(1) << n : 0) - 1);
            plan.resize(size_t(1 + R * H));
            const int c = sparsp::plan_chunks(g, demand.data(), R, rank, in(1, H), in(1, H),
                                              plan.data(), int(plan.size()));
            if (c < 1) ++failures;
            plan.resize(size_t(c));
        } else {  // anything the entry point accepts: gaps, empty ranges, overlaps, any order
            for (int k = in(0, 6); k > 0; --k) {
                const int lo = in(0, n), h0 = in(0, H - 1);
                plan.push_back({0, lo, in(lo, n), h0, in(h0 + 1, H), 0});
            }
        }
        std::vector<int> want(size_t(H) * n, 0), got(want);
        bool twice = false;
        for (const auto& c : plan)
            for (int h = c.head_begin; h < c.head_end; ++h)
                for (int j = c.kv_blk_begin; j < c.kv_blk_end; ++j)
                    twice = ++want[size_t(h) * n + j] > 1 || twice;
        std::vector<sparsp::AttnPart> launches;
        std::vector<std::pair<int, int>> empty;
        const bool ok = sparsp::merge_chunks(H, plan.data(), int(plan.size()), &launches, &empty);
        if (ok == twice) ++failures;
        if (!ok) { ++refused; continue; }
        ++merged;
        std::vector<int> state(size_t(H), 0);  // 0 nothing, 1 written, 2 cleared
        for (const auto& p : launches)
            for (int h = p.h_lo; h < p.h_hi; ++h) {
                if ((p.acc != 0) != (state[h] == 1)) ++failures;
                state[h] = 1;
                for (int j = p.kv_lo; j < p.kv_hi; ++j) ++got[size_t(h) * n + j];
            }
        for (const auto& e : empty)
            for (int h = e.first; h < e.second; ++h) {
                if (state[h]) ++failures;
                state[h] = 2;
            }
        for (int h = 0; h < H; ++h)
            if (!state[h]) ++failures;
        if (got != want) ++failures;
        if (it % 4 == 0 && launches.size() == 1 && launches[0].kv_lo == 0 && launches[0].kv_hi == n)
            ++single;
        else if (it % 4 == 0)
            ++failures;  // a schedule is one launch over everything
    }
    printf("%d merged, %d refused, %d schedules in one launch, %d failures\n", merged, refused,
           single, failures);
    return failures ? 1 : 0;
}
