// Pure host code of libsparsp: the shard-by-shard schedule (Section 2.3,
// Section 7), Eq. 4's placed order of the blocks (Section 4.3), the Eq. 3
// block count and the routing volumes of Section 5.1. Nothing here touches a
// device; the descriptions of each rule sit with their launch-side
// counterparts in chunks.hip and placement.hip.
#include <algorithm>
#include <map>
#include <vector>

#include "sparsp_launch.h"

namespace sparsp {

int plan_chunks(const Geom& g, const uint64_t* demand, int ranks, int rank, int heads_per_chunk,
                int tail_heads_per_chunk, sparsp_chunk* out, int max_chunks) {
    auto count = [&](int h0, int h1, int lo, int hi) {
        int c = 0;
        for (int h = h0; h < h1; ++h)
            for (int j = lo; j < hi; ++j) c += int((demand[int64_t(h) * g.W + (j >> 6)] >> (j & 63)) & 1);
        return c;
    };
    auto shard = [&](int p, int* lo, int* hi) {
        *lo = int(int64_t(p) * g.n / ranks);
        *hi = int(int64_t(p + 1) * g.n / ranks);
    };
    std::vector<sparsp_chunk> plan;
    int lo, hi;
    shard(rank, &lo, &hi);
    plan.push_back({rank, lo, hi, 0, g.H, count(0, g.H, lo, hi)});
    for (int k = 1; k < ranks; ++k) {
        const int p = (rank + k) % ranks;
        shard(p, &lo, &hi);
        const int size = k == ranks - 1 ? tail_heads_per_chunk : heads_per_chunk;
        std::vector<sparsp_chunk> part;
        for (int h0 = 0; h0 < g.H; h0 += size) {
            const int h1 = std::min(g.H, h0 + size);
            part.push_back({p, lo, hi, h0, h1, count(h0, h1, lo, hi)});
        }
        std::stable_sort(part.begin(), part.end(), [](const sparsp_chunk& a, const sparsp_chunk& b) {
            return a.blocks != b.blocks ? a.blocks > b.blocks : a.head_begin < b.head_begin;
        });
        plan.insert(plan.end(), part.begin(), part.end());
    }
    if (int(plan.size()) > max_chunks) return -int(plan.size());
    std::copy(plan.begin(), plan.end(), out);
    return int(plan.size());
}

std::vector<ChunkStep> chunk_steps(int H, const sparsp_chunk* plan, int n_chunks) {
    struct Group {
        int lo, hi;
        std::vector<char> has;  // per head
    };
    std::vector<Group> groups;
    std::map<std::pair<int, int>, std::vector<int>> of_range;  // groups of a block range, ascending
    std::vector<int> last(H, -1);  // the latest group of each head
    for (int c = 0; c < n_chunks; ++c) {
        const sparsp_chunk& ch = plan[c];
        if (ch.kv_blk_begin >= ch.kv_blk_end) continue;  // no block, nothing to add
        const int after = *std::max_element(last.begin() + ch.head_begin, last.begin() + ch.head_end);
        std::vector<int>& same = of_range[{ch.kv_blk_begin, ch.kv_blk_end}];
        auto it = std::upper_bound(same.begin(), same.end(), after);
        int k;
        if (it != same.end()) {
            k = *it;
        } else {
            k = int(groups.size());
            groups.push_back({ch.kv_blk_begin, ch.kv_blk_end, std::vector<char>(H, 0)});
            same.push_back(k);
        }
        for (int h = ch.head_begin; h < ch.head_end; ++h) {
            groups[k].has[h] = 1;
            last[h] = k;
        }
    }
    std::vector<ChunkStep> steps;
    std::vector<char> seen(H, 0);  // heads whose rows hold a result
    auto clear = [&](int h_lo, int h_hi) {  // the heads of [h_lo, h_hi) without one
        for (int h = h_lo; h < h_hi;) {
            int e = h;
            while (e < h_hi && !seen[e]) ++e;
            if (e > h) steps.push_back({true, AttnPart{0, 0, h, e, 0}});
            h = e + 1;
        }
    };
    for (const Group& g : groups) {
        for (int h = 0; h < H;) {
            int e = h, old = 0;
            while (e < H && g.has[e]) old += seen[e++];
            if (e > h) {
                if (old > 0 && old < e - h) clear(h, e);  // all of a launch folds in, or none
                steps.push_back({false, AttnPart{g.lo, g.hi, h, e, old > 0 ? 1 : 0}});
                std::fill(seen.begin() + h, seen.begin() + e, 1);
            }
            h = e + 1;
        }
    }
    clear(0, H);
    return steps;
}

void periodic_placement(int L, int block, int frame_tokens, int ranks, int32_t* perm,
                        int32_t* rank_begin) {
    const int n = (L + block - 1) / block;
    std::vector<int> owner(n);
    for (int j = 0; j < n; ++j)
        owner[j] = int(int64_t(ranks) * ((int64_t(j) * block) % frame_tokens) / frame_tokens);
    if (L % block) owner[n - 1] = ranks - 1;
    int k = 0;
    for (int p = 0; p < ranks; ++p) {
        rank_begin[p] = k;
        for (int j = 0; j < n; ++j)
            if (owner[j] == p) perm[k++] = j;
    }
    rank_begin[ranks] = k;
}

void remote_demand(const Geom& g, const uint64_t* demand, int64_t* remote, int64_t* demanded) {
    int64_t rem = 0, all = 0;
    for (int h = 0; h < g.H; ++h)
        for (int j = 0; j < g.n; ++j) {
            if (!((demand[int64_t(h) * g.W + (j >> 6)] >> (j & 63)) & 1)) continue;
            ++all;
            if (j < g.i0 || j >= g.i1) ++rem;
        }
    *remote = rem;
    *demanded = all;
}

void route_volume(const Geom& g, const uint64_t* demands, int ranks, int producer, int64_t* dense,
                  int64_t* relay, int64_t* direct) {
    const int lo = int(int64_t(producer) * g.n / ranks), hi = int(int64_t(producer + 1) * g.n / ranks);
    int64_t rel = 0, dir = 0;
    std::vector<uint64_t> down(g.W);
    for (int h = 0; h < g.H; ++h) {
        std::fill(down.begin(), down.end(), 0);
        for (int k = ranks - 1; k >= 1; --k) {  // farthest consumer first: down = union of distance >= k
            const int c = (producer + k) % ranks;
            const uint64_t* dm = demands + (int64_t(c) * g.H + h) * g.W;
            for (int j = lo; j < hi; ++j) {
                const uint64_t bit = uint64_t(1) << (j & 63);
                if (dm[j >> 6] & bit) {
                    ++dir;
                    down[j >> 6] |= bit;
                }
            }
            for (int j = lo; j < hi; ++j) rel += int64_t((down[j >> 6] >> (j & 63)) & 1);
        }
    }
    *dense = int64_t(ranks - 1) * g.H * (hi - lo);
    *relay = rel;
    *direct = dir;
}

}  // namespace sparsp
