// Host side of shard-by-shard attention (Section 2.3, Section 7): running a
// plan. The plan itself (plan_chunks, in host_plan.cpp) orders the work of rank r
// over the owners' KV shards:
//   * shard p holds the blocks [floor(p n / R), floor((p+1) n / R));
//   * the local shard (p = r) comes first and stays whole: one chunk with all
//     heads (Section 7.1: it needs no transfer);
//   * the remote shards follow in ring order r+1, ..., r+R-1 (mod R), each cut
//     into runs of heads_per_chunk consecutive heads, the last remote shard
//     into finer runs of tail_heads_per_chunk heads (Section 7.1: the final
//     block of the pipeline is chunked finer to shorten the drain);
//   * inside each remote shard, chunks run by selected blocks descending, then
//     head ascending (Section 7.2: the sparsest chunk goes last, so the
//     computation left exposed after the last transfer is the smallest).
// A chunk's selected blocks are its heads' demanded blocks inside the shard,
// counted from the demand bitsets.
//
// run_chunks executes a plan on one stream. Everything the plan reads is in
// place when the call's work starts (the call is stream-ordered), so the chunks
// need not be launches of their own: the chunks of one shard are one step over all
// their heads (chunk_steps), and in bf16 the steps over the same heads are one launch,
// each row taking its shards one after another. A head still folds its shards in plan
// order through the log-sum-exp inside the attention kernel, each with a softmax of its
// own, so the result has the rounding of a chunk-by-chunk run; shards with no kept
// block of a row cost it the look at its list. One launch per chunk leaves the GPU to
// the longest row of each of a few heads, and one per shard to the longest of each
// shard: 40 heads x 147 rows, 591 blocks of 128, 89 kept, four owners, 31 chunks took
// 6.84 ms, four launches 4.75 ms, one 4.25 ms. (One softmax for all shards would take
// 3.80 ms, but then fewer top probabilities are exact: error of O against 64 bits
// 6.4e-4 instead of 6.3e-4.) Heads that no chunk covers end as the empty result.
#include <new>

#include "sparsp_internal.h"

namespace sparsp {
namespace {

struct Run {  // the arguments every launch of a plan shares
    const Geom& g;
    const void* Q;
    const int32_t* sel;
    int keep;
    const int32_t* slot_of;
    const void *Kp, *Vp;
    int64_t capacity;
    float scale;
    float *O, *lse;
    hipStream_t s;

    hipError_t attend(const AttnPart& part) const {
        return g.bf16 ? launch_attn_bf16(g, Q, sel, keep, slot_of, Kp, Vp, capacity, scale, part, O,
                                         false, lse, s)
                      : launch_attn_f32(g, (const float*)Q, sel, keep, slot_of, (const float*)Kp,
                                        (const float*)Vp, capacity, scale, part, O, lse, s);
    }
    hipError_t clear(int h_lo, int h_hi) const {  // the empty result for a run of heads
        const int64_t rows = int64_t(g.nq) * g.block;
        return launch_fill_identity(O + h_lo * rows * g.d, lse + h_lo * rows, (h_hi - h_lo) * rows,
                                    g.d, s);
    }
};

}  // namespace

hipError_t run_chunks(const Geom& g, const void* Q, const int32_t* sel, int keep,
                      const int32_t* slot_of, const void* Kp, const void* Vp, int64_t capacity,
                      float scale, const sparsp_chunk* plan, int n_chunks, float* O, float* lse,
                      hipStream_t s) {
    const Run run{g, Q, sel, keep, slot_of, Kp, Vp, capacity, scale, O, lse, s};
    try {
        const std::vector<ChunkStep> steps = chunk_steps(g.H, plan, n_chunks);
        for (size_t i = 0; i < steps.size();) {
            AttnPart part = steps[i].part;
            if (steps[i].clear) {
                if (hipError_t e = run.clear(part.h_lo, part.h_hi); e != hipSuccess) return e;
                ++i;
                continue;
            }
            // The steps that follow over the same heads, in one launch. (A part of all
            // blocks stays alone: it may be a kernel of its own.)
            const bool joins = g.bf16 && part.kv_hi - part.kv_lo < g.n;
            Shards& sh = part.shards;
            do {
                sh.lo[sh.n] = steps[i].part.kv_lo;
                sh.hi[sh.n++] = steps[i++].part.kv_hi;
            } while (joins && sh.n < kMaxShards && i < steps.size() && !steps[i].clear &&
                     steps[i].part.acc && steps[i].part.h_lo == part.h_lo &&
                     steps[i].part.h_hi == part.h_hi);
            if (hipError_t e = run.attend(part); e != hipSuccess) return e;
        }
    } catch (const std::bad_alloc&) {  // no exception may leave the C entry
        return hipErrorOutOfMemory;
    }
    return hipSuccess;
}

}  // namespace sparsp
