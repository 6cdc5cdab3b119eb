// Random chunk plans, well formed and not: the launches of chunk_steps must take
// every head through its chunks' block ranges in plan order, write a head before
// folding into it, never mix the two in a launch, leave exactly the uncovered heads
// cleared, and never be more than the plan's chunks; a schedule of plan_chunks takes
// one launch per shard.
#include <cstdio>
#include <random>
#include <set>

#include "../../paper_2609_32197_amd/csrc/sparsp_launch.h"

int main() {
    std::mt19937 rng(7);
    auto in = [&](int lo, int hi) { return lo + int(rng() % unsigned(hi - lo + 1)); };
    int failures = 0, chunks = 0, launches = 0;
    for (int it = 0; it < 20000; ++it) {
        const int H = in(1, 9), n = in(1, 40);
        int shards = -1;
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
            shards = R;
        } else if (it % 4 == 1) {  // a local chunk of all heads, then one of some heads each
            const int mid = in(1, n);
            plan.push_back({0, 0, mid, 0, H, 0});
            for (int h = 0; h < H; ++h)
                if (rng() % 2) plan.push_back({1, mid, n, h, h + 1, 0});
        } else {  // anything the entry point accepts: gaps, empty ranges, overlaps, any order
            std::vector<std::pair<int, int>> ranges;
            for (int k = in(1, 4); k > 0; --k) {
                const int lo = in(0, n);
                ranges.push_back({lo, in(lo, n)});
            }
            for (int k = in(0, 8); k > 0; --k) {
                const auto& r = ranges[size_t(in(0, int(ranges.size()) - 1))];
                const int h0 = in(0, H - 1);
                plan.push_back({0, r.first, r.second, h0, in(h0 + 1, H), 0});
            }
        }
        std::vector<std::vector<std::pair<int, int>>> want(static_cast<size_t>(H)), got(want);
        for (const auto& c : plan)
            for (int h = c.head_begin; h < c.head_end; ++h)
                if (c.kv_blk_begin < c.kv_blk_end)
                    want[size_t(h)].push_back({c.kv_blk_begin, c.kv_blk_end});
        int attends = 0;
        std::vector<char> state(size_t(H), 0);  // 1: holds a result
        for (const auto& step : sparsp::chunk_steps(H, plan.data(), int(plan.size()))) {
            const sparsp::AttnPart& p = step.part;
            if (p.h_lo < 0 || p.h_hi > H || p.h_lo >= p.h_hi) { ++failures; break; }
            attends += !step.clear;
            for (int h = p.h_lo; h < p.h_hi; ++h) {
                if (step.clear) {
                    if (!got[size_t(h)].empty() || state[size_t(h)]) ++failures;
                } else {
                    if ((p.acc != 0) != (state[size_t(h)] != 0)) ++failures;
                    got[size_t(h)].push_back({p.kv_lo, p.kv_hi});
                }
                state[size_t(h)] = 1;
            }
        }
        if (got != want) ++failures;
        for (char s : state)
            if (!s) ++failures;
        if (attends > int(plan.size())) ++failures;
        if (shards >= 0) {
            std::set<std::pair<int, int>> ranges;
            for (const auto& c : plan) ranges.insert({c.kv_blk_begin, c.kv_blk_end});
            if (attends != int(ranges.size()) || attends > shards) ++failures;
        }
        chunks += int(plan.size());
        launches += attends;
    }
    printf("%d chunks in %d launches, %d failures\n", chunks, launches, failures);
    return failures ? 1 : 0;
}
