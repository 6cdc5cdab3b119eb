// Step 4, float32: block-sparse attention for float32 inputs (Eq. 1 over the
// kept blocks, softmax renormalised over the kept keys, online).
//
// This is the precision path: every product and sum is float32, on the matrix
// cores (v_mfma_f32_16x16x4_f32: float32 in, float32 accumulation), which
// keeps the result within 1e-5 of the float64 definition at the sizes it
// serves.
//
// Work split. A workgroup takes 16 * NQ queries of one (head, local query
// block) row and all of the row's kept keys. Its KW waves share the queries
// and split the keys: wave w takes the 16-key tiles w, w + KW, ... of the kept
// list and runs its own online softmax over them; the KW partial results are
// merged at the end through their maxima and sums (the online-softmax merge of
// Section 2.3). Small grids thus still put several waves on every row, and no
// barrier stands inside the loop.
//
// Products are computed transposed, S^T = K Q^T and O^T = V^T P^T. The four
// products of a 16-wide d chunk take their k values in an order of our own: in
// step t of chunk c the lanes of group g = lane / 16 supply element 16 c + 4 g
// + t, so each lane takes its share of a chunk as one float4, of K [block, d]
// and Q alike. The scores then sit as P^T operands already (lane: query lane %
// 16, keys 4 g .. +3), and a float4 of a V^T row holds exactly a lane's keys,
// so neither operand is shuffled.
//
// Tiles. Each wave stages its own tiles (16 keys of K, the same 16 of V^T) in
// its own LDS with direct-to-LDS buffer loads, K of the next tile while the
// output product of this one runs, V of the next during the next scores; it
// waits for its own copies by count and never for another wave. One copy
// instruction moves 16 rows of 64 bytes, four neighbouring lanes a row, because
// the vector cache looks up one line per row and quarter-wave: the same operands
// read straight into registers, 16 rows of 16 bytes per quarter-wave, took four
// times the lookups and held the kernel at 98 TFLOP/s (H = 8, d = 128, 1,024
// rows of 128 queries, 32 blocks kept). The four 16-byte chunks of a row are
// rotated by its index, which makes the operand reads free of bank conflicts.
#include "sparsp_internal.h"

namespace sparsp {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
// The running max moves once a score exceeds it by this much (log2 units):
// probabilities stay below 2^8, and float32 loses nothing by the offset.
constexpr float kRescale = 8.0f;

// Max and sum over the four lanes l, l^16, l^32, l^48 that share a query: a
// swap with x in both operands returns the pair {x[l], x[l^16]} (then l^32).
__device__ __forceinline__ float quad_max(float x) {
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float quad_sum(float x) {
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

// s_waitcnt vmcnt(n), leaving the other counters alone.
template <int N>
__device__ __forceinline__ void wait_vmem() {
    static_assert(N >= 0 && N < 16, "vmcnt field");
    __builtin_amdgcn_s_waitcnt(0x0F70 | N);
}

// Direct-to-LDS copy of one tile, DC instructions of 1 KB, to the LDS byte
// address `lds` on. `base` and `bytes` describe the memory from the tile's
// start to the end of its slot: what lies past that reads as zero. In inline
// assembly because the compiler would otherwise wait for every copy in flight
// before any LDS read; M0 is restored, and a wait state follows each write.
template <int DC>
__device__ __forceinline__ void copy_tile(const float* base, uint32_t bytes, uint32_t lds,
                                          const int (&voff)[DC]) {
#if defined(__HIP_DEVICE_COMPILE__)
    const uint64_t b = reinterpret_cast<uint64_t>(base);
    u32x4_t desc;
    desc.x = __builtin_amdgcn_readfirstlane(uint32_t(b));
    desc.y = __builtin_amdgcn_readfirstlane(uint32_t(b >> 32) & 0xffffu);  // stride 0
    desc.z = __builtin_amdgcn_readfirstlane(bytes);                        // num_records
    desc.w = 0x00020000u;
#pragma unroll
    for (int c = 0; c < DC; ++c) {
        uint32_t saved;
        asm volatile(
            "s_mov_b32 %[sv], m0\n\ts_mov_b32 m0, %[lds]\n\ts_nop 0\n\t"
            "buffer_load_dwordx4 %[o], %[desc], 0 offen lds\n\ts_mov_b32 m0, %[sv]"
            : [sv] "=&s"(saved)
            : [lds] "s"(lds + 1024u * c), [desc] "s"(desc), [o] "v"(voff[c])
            : "memory");
    }
#endif
}

// LDS of a workgroup: per wave a K and a V tile of DC KB each, then the kept
// list; after the loop the partial results in their place (per wave: 4 DC NQ
// registers of 64 lanes, and max and sum per query).
__host__ __device__ constexpr int merge_floats(int DC, int NQ) {
    return DC * NQ * 4 * 64 + 2 * 16 * NQ;
}

constexpr int kCus = 256;  // of an MI355X
constexpr int kPastSlot = 1 << 30;  // a byte offset past every slot (256 x 128 x 4 at most)

// DC: 16-wide chunks of d (d <= 16 DC); NQ: 16-query groups per wave.
template <int DC, int NQ>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2))) void attn_f32_kernel(
    const float* __restrict__ Q, const int32_t* __restrict__ sel, const int32_t* __restrict__ slot_of,
    const float* __restrict__ Kp, const float* __restrict__ Vp, float* __restrict__ O,
    float* __restrict__ lse, int L, int n, int d, int block, int i0, int nq, int keep,
    int64_t capacity, float c2 /* scale * log2(e) */, int kv_lo, int kv_hi, int h_lo, int acc,
    const int32_t* __restrict__ order, int rows, int parts /* workgroups per row */,
    int first, int count /* this launch's rows, or positions of the order */) {
    extern __shared__ __attribute__((aligned(16))) int32_t smem[];
    __shared__ int wave_cnt[8];
    const int tid = threadIdx.x, nthr = blockDim.x, KW = nthr >> 6;
    // slot of each usable kept entry; bit 31: the partial last block
    int32_t* codes = smem + KW * 2 * DC * 256;
    const int lane = tid & 63, qi = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Workgroup -> (row, part of its queries). Consecutive workgroups go to the
    // eight XCDs in turn; an XCD gets a contiguous range of rows, whose kept
    // blocks overlap and then hit in its L2. With an explicit row order (e.g.
    // longest first) positions x, x + 8, ... of the order go to XCD x.
    const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
    int row, part;
    if (order) {
        const int pos = (idx / parts) * 8 + xcd;
        part = idx % parts;
        if (pos >= count) return;
        row = order[first + pos];
        if (row < 0 || row >= rows) return;
    } else {
        const int total = count * parts, per = total >> 3, rem = total & 7;
        const int w = xcd * per + min(xcd, rem) + idx;
        row = first + w / parts;
        part = w % parts;
    }
    const int q0 = part * 16 * NQ;  // first query of the block for this workgroup
    const int h = h_lo + row / nq, r = row % nq;

    // The kept list: usable entries inside [kv_lo, kv_hi), in list order.
    int nkeep = 0;
    {
        const int32_t* srow = sel + (int64_t(h) * nq + r) * keep;
        const int32_t* hslot = slot_of + int64_t(h) * n;
        const bool ragged = (L % block) != 0;
        for (int base = 0; base < keep; base += nthr) {
            const int jj = base + tid;
            int slot = -1, j = -1;
            if (jj < keep) {
                j = srow[jj];
                if (j >= kv_lo && j < kv_hi && j >= 0 && j < n) {
                    slot = hslot[j];
                    if (slot >= capacity) slot = -1;
                }
            }
            const uint64_t bal = __ballot(slot >= 0);
            if (lane == 0) wave_cnt[wave] = __popcll(bal);
            __syncthreads();
            int off = nkeep, total = 0;
            for (int w = 0; w < KW; ++w) {
                off += w < wave ? wave_cnt[w] : 0;
                total += wave_cnt[w];
            }
            const int below = __builtin_amdgcn_mbcnt_hi(
                uint32_t(bal >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(bal), 0));
            if (slot >= 0) codes[off + below] = slot | ((ragged && j == n - 1) ? INT32_MIN : 0);
            nkeep += total;
            __syncthreads();
        }
    }
    if (acc && nkeep == 0) return;  // nothing to fold in
    const int last_cnt = L - (L / block) * block;  // valid keys of a partial last block

    // Q^T operands. Elements past d are zero, as they are in the K operand.
    floatx4 qf[NQ][DC];
    bool qvalid[NQ];
#pragma unroll
    for (int a = 0; a < NQ; ++a) {
        const int qrow = q0 + 16 * a + qi;
        const int64_t qtok = int64_t(i0 + r) * block + qrow;
        qvalid[a] = qrow < block && qtok < L;
#pragma unroll
        for (int c = 0; c < DC; ++c) {
            const int e = 16 * c + 4 * g;
            qf[a][c] = (qvalid[a] && e < d)
                           ? *reinterpret_cast<const floatx4*>(Q + (int64_t(h) * L + qtok) * d + e)
                           : floatx4{};
        }
    }

    floatx4 o[NQ][DC];
    float m[NQ], l[NQ], lim[NQ];         // lim: where m moves, kRescale above it
    float off[NQ];                       // m, or 0 while the query has no score above -inf
    const float slack = kRescale / c2;  // in unscaled scores
#pragma unroll
    for (int a = 0; a < NQ; ++a) {
        m[a] = lim[a] = -INFINITY;
        l[a] = off[a] = 0.f;
#pragma unroll
        for (int c = 0; c < DC; ++c) o[a][c] = floatx4{};
    }

    // Copy offsets: lane 4 i + p of instruction c brings row i (a key of K, a
    // dim 16 c + i of V^T), chunk p ^ (i / 4) of its four. A chunk past d would be the
    // next key's: it is asked for past the end of the slot, which reads as zero (an
    // infinite value times the query's zero would be NaN).
    const float* lk = reinterpret_cast<const float*>(smem) + wave * 2 * DC * 256;
    const float* lv = lk + DC * 256;
    const uint32_t lk_at = uint32_t(reinterpret_cast<uintptr_t>(lk));
    const uint32_t lv_at = uint32_t(reinterpret_cast<uintptr_t>(lv));
    int koff[DC], voff[DC];
    {
        const int i = lane >> 2, p = (lane & 3) ^ ((lane >> 4) & 3);
#pragma unroll
        for (int c = 0; c < DC; ++c) {
            koff[c] = 16 * c + 4 * p < d ? (i * d + 16 * c + 4 * p) * 4 : kPastSlot;
            voff[c] = ((16 * c + i) * block + 4 * p) * 4;
        }
    }
    const int at = (qi * 4 + (g ^ (qi >> 2))) * 4;  // this lane's float4 of a 1 KB piece
    const uint32_t slot_bytes = uint32_t(block) * uint32_t(d) * 4u;
    auto copy_k = [&](int code, int tt) {  // rows past the valid keys read as zero
        const uint32_t off = uint32_t(16 * tt) * uint32_t(d);
        const uint32_t rows_left = uint32_t((code < 0 ? last_cnt : block) - 16 * tt);
        copy_tile<DC>(Kp + int64_t(code & INT32_MAX) * block * d + off,
                      rows_left * uint32_t(d) * 4u, __builtin_amdgcn_readfirstlane(lk_at), koff);
    };
    auto copy_v = [&](int code, int tt) {
        copy_tile<DC>(Vp + int64_t(code & INT32_MAX) * block * d + 16 * tt,
                      slot_bytes - 64u * uint32_t(tt), __builtin_amdgcn_readfirstlane(lv_at), voff);
    };

    // Tiles of 16 keys: tile t of entry e covers keys 16 t .. of its block.
    const int nt = (block + 15) >> 4;
    int e = 0, t = wave, code = 0;
    auto settle = [&]() {  // (e, t) to the next tile that holds a valid key
        for (;;) {
            while (t >= nt) {
                t -= nt;
                ++e;
            }
            if (e >= nkeep) return;
            code = __builtin_amdgcn_readfirstlane(codes[e]);
            if (16 * t < (code < 0 ? last_cnt : block)) return;
            t += KW;
        }
    };

    settle();
    wait_vmem<0>();  // from here on only the copies below are in flight
    if (e < nkeep) copy_k(code, t);
    while (e < nkeep) {
        const int kn = (code < 0 ? last_cnt : block) - 16 * t;  // valid keys of the tile, >= 1
        copy_v(code, t);
        wait_vmem<DC>();  // K landed; V may still be in flight
        __builtin_amdgcn_sched_barrier(0);
        // Scores: lane holds keys 4 g .. +3 of query qi. Two chains per query
        // group, so that no product waits on the one before it.
        floatx4 s[NQ][2];
#pragma unroll
        for (int a = 0; a < NQ; ++a) s[a][0] = s[a][1] = floatx4{};
#pragma unroll
        for (int c = 0; c < DC; ++c) {
            const floatx4 kf = *reinterpret_cast<const floatx4*>(lk + c * 256 + at);
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int a = 0; a < NQ; ++a)
                    s[a][u & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[u], qf[a][c][u],
                                                                       s[a][u & 1], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        // The next tile's K (the last tile's is read again rather than none, so
        // that the count of copies in flight is the same in every iteration).
        const int cur_code = code, cur_t = t;
        t += KW;
        settle();
        const bool more = e < nkeep;
        copy_k(more ? code : cur_code, more ? t : cur_t);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int a = 0; a < NQ; ++a) {
            // Scores stay unscaled, the running max m too, and only their differences
            // are scaled: the top probability is exactly 1 at any scale, and a key's
            // rounding grows with its distance from the max, not with the score. (A
            // scaled max, rounded, against fma(x, c2, -max): from scores of about 2^31
            // on, the difference of the two roundings leaves the exponent's range.)
            floatx4 x = s[a][0] + s[a][1];
            if (kn < 16) {
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (4 * g + u >= kn) x[u] = -INFINITY;
            }
            const float mx = quad_max(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])));
            if (__ballot(mx > lim[a]) != 0) {
                const float m_new = fmaxf(m[a], mx);
                const float to = m_new == -INFINITY ? 0.f : m_new;
                const float alpha = __builtin_amdgcn_exp2f((m[a] - to) * c2);
                m[a] = m_new;
                off[a] = to;
                lim[a] = m_new + slack;
                l[a] *= alpha;
#pragma unroll
                for (int c = 0; c < DC; ++c) o[a][c] *= alpha;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                s[a][0][u] = __builtin_amdgcn_exp2f((x[u] - off[a]) * c2);
                l[a] += s[a][0][u];
            }
        }
        wait_vmem<DC>();  // V landed; the next K may still be in flight
        __builtin_amdgcn_sched_barrier(0);
        if (kn < 16) {  // what stands past the valid keys must not meet their zero weights
            float* mine = const_cast<float*>(lv) + at;
#pragma unroll
            for (int c = 0; c < DC; ++c)
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (4 * g + u >= kn) mine[c * 256 + u] = 0.f;
        }
        // two d chunks at a time, so that successive products are independent
#pragma unroll
        for (int c0 = 0; c0 < DC; c0 += 2) {
            floatx4 vf[2];
#pragma unroll
            for (int c = c0; c < c0 + 2 && c < DC; ++c)
                vf[c - c0] = *reinterpret_cast<const floatx4*>(lv + c * 256 + at);
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int c = c0; c < c0 + 2 && c < DC; ++c)
#pragma unroll
                    for (int a = 0; a < NQ; ++a)
                        o[a][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[c - c0][u], s[a][0][u],
                                                                       o[a][c], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    wait_vmem<0>();  // the last copy may not land in what follows

    // Merge of the waves' partial softmaxes: weight each by 2^(m_w - M) for the
    // query's max M (0 for a wave that saw no key), then sum. Every wave leaves
    // its registers in LDS; wave w then finishes the d chunks w, w + KW, ...
    // With acc, every lane reads the stored lse before the barrier that lets
    // one of them rewrite it.
    const int64_t orow0 = (int64_t(h) * nq + r) * block + q0;
    float l_old[NQ];
#pragma unroll
    for (int a = 0; a < NQ; ++a) {
        const int qrow = 16 * a + qi;
        l_old[a] = (acc && q0 + qrow < block) ? lse[orow0 + qrow] : -INFINITY;
    }
    __syncthreads();  // every wave is done with its tiles and the kept list
    float* area = reinterpret_cast<float*>(smem);
    constexpr int STRIDE = merge_floats(DC, NQ);
    {
        float* mine = area + wave * STRIDE;
#pragma unroll
        for (int a = 0; a < NQ; ++a) {
#pragma unroll
            for (int c = 0; c < DC; ++c)
                *reinterpret_cast<floatx4*>(mine + ((a * DC + c) * 64 + lane) * 4) = o[a][c];
            const float ls = quad_sum(l[a]);
            if (g == 0) {
                mine[DC * NQ * 256 + (2 * a) * 16 + qi] = m[a];
                mine[DC * NQ * 256 + (2 * a + 1) * 16 + qi] = ls;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int a = 0; a < NQ; ++a) {
        const int qrow = 16 * a + qi;
        float M = -INFINITY;
        for (int w = 0; w < KW; ++w) M = fmaxf(M, area[w * STRIDE + DC * NQ * 256 + 2 * a * 16 + qi]);
        float tot = 0.f, wt[8];
#pragma unroll
        for (int w = 0; w < 8; ++w) {
            wt[w] = 0.f;
            if (w < KW) {
                const float* st = area + w * STRIDE + DC * NQ * 256 + 2 * a * 16 + qi;
                wt[w] = st[0] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((st[0] - M) * c2);
                tot += wt[w] * st[16];
            }
        }
        const bool live = qvalid[a] && tot > 0.f;
        const float inv = live ? 1.0f / tot : 0.f;
        // Folding into a running result: the stored row weighs ka, this part kb.
        float ka = 0.f, kb = inv;
        const float lb2 = fmaf(M, c2, log2f(tot));  // this part's log-sum-exp, log2 units
        float lse_out = live ? lb2 * kLn2 : -INFINITY;
        bool store = q0 + qrow < block;
        if (acc) {
            store = store && live;  // a row with no key in this part is left as it is
            if (live) {
                const float la2 = l_old[a] * kLog2e;
                const float mm = fmaxf(la2, lb2);
                const float wa = la2 == -INFINITY ? 0.f : exp2f(la2 - mm);
                const float wb = exp2f(lb2 - mm);
                ka = wa / (wa + wb);
                kb = wb / (wa + wb) * inv;
                lse_out = (mm + log2f(wa + wb)) * kLn2;
            }
        }
        if (!store) continue;
        for (int c = wave; c < DC; c += KW) {
            floatx4 x = {};
#pragma unroll
            for (int w = 0; w < 8; ++w)
                if (w < KW)
                    x += wt[w] * *reinterpret_cast<const floatx4*>(area + w * STRIDE +
                                                                   ((a * DC + c) * 64 + lane) * 4);
            const int e0 = 16 * c + 4 * g;
            if (e0 >= d) continue;
            floatx4* op = reinterpret_cast<floatx4*>(O + (orow0 + qrow) * d + e0);
            floatx4 y = live ? kb * x : floatx4{};
            if (acc) y += ka * *op;
            *op = y;
        }
        if (lse && wave == 0 && g == 0) lse[orow0 + qrow] = lse_out;
    }
}

template <int DC>
hipError_t launch_dc(const Geom& g, const float* Q, const int32_t* sel, int keep,
                     const int32_t* slot_of, const float* Kp, const float* Vp, int64_t capacity,
                     float c2, const AttnPart& part, float* O, float* lse, hipStream_t s) {
    const int G = (part.h_hi - part.h_lo) * g.nq;
    // Two query groups per wave feed each operand read to twice the products;
    // one makes finer workgroups and pads a block of, say, 100 queries to 112
    // instead of 128. The fuller CU sets the time, so the two are compared by
    // the 16-query groups that one CU gets at most, with two groups per wave
    // worth 8%. Measured (us, one group / two): 12 heads x 25 rows of 64
    // queries, d = 96 98 / 104; 3 x 214 rows of 100, d = 96 399 / 438; 6 x 19
    // rows of 100, d = 128 179 / 165; 8 x 128 rows of 128, d = 128 2,356 /
    // 2,128; 14 x 169 rows of 64, d = 64 459 / 428.
    const int w1 = G * ((g.block + 15) / 16), w2 = G * ((g.block + 31) / 32);
    const int per1 = (w1 + kCus - 1) / kCus, per2 = 2 * ((w2 + kCus - 1) / kCus);
    const int nqg = 12 * per2 <= 13 * per1 ? 2 : 1;
    // Four waves split the keys; eight where every CU has one workgroup at most
    // (2 x 16 rows of 64, d = 64: 9.7 against 10.5 us; elsewhere 4 to 28% slower).
    const int kw = nqg == 1 && w1 <= kCus ? 8 : 4;
    const int parts = (g.block + 16 * nqg - 1) / (16 * nqg);
    const size_t dyn = max(size_t(kw) * 2 * DC * 1024 + size_t(keep) * 4,
                           size_t(kw) * merge_floats(DC, nqg) * 4);
    auto* kern = nqg == 2 ? attn_f32_kernel<DC, 2> : attn_f32_kernel<DC, 1>;
    // A launch holds less than 2^32 threads, which 270 million queries in parts of 16
    // (four waves each) would pass: such a call takes several launches.
    const int most = int((UINT32_MAX / (64u * kw * parts)) & ~7u);
    for (int first = 0; first < G; first += most) {
        const int count = min(most, G - first);
        const int grid = part.order ? (count + 7) / 8 * 8 * parts : count * parts;
        kern<<<grid, 64 * kw, dyn, s>>>(Q, sel, slot_of, Kp, Vp, O, lse, g.L, g.n, g.d, g.block,
                                        g.i0, g.nq, keep, capacity, c2, part.kv_lo, part.kv_hi,
                                        part.h_lo, part.acc, part.order, G, parts, first, count);
        if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

hipError_t launch_attn_f32(const Geom& g, const float* Q, const int32_t* sel, int keep,
                           const int32_t* slot_of, const float* Kp, const float* Vp,
                           int64_t capacity, float scale, const AttnPart& part, float* O,
                           float* lse, hipStream_t s) {
    (void)hipGetLastError();
    const float c2 = scale * kLog2e;
#define SPARSP_F32_LAUNCH(DC)                                                                 \
    return launch_dc<DC>(g, Q, sel, keep, slot_of, Kp, Vp, capacity, c2, part, O, lse, s)
    switch ((g.d + 15) / 16) {
        case 1: SPARSP_F32_LAUNCH(1);
        case 2: SPARSP_F32_LAUNCH(2);
        case 3: SPARSP_F32_LAUNCH(3);
        case 4: SPARSP_F32_LAUNCH(4);
        case 5: SPARSP_F32_LAUNCH(5);
        case 6: SPARSP_F32_LAUNCH(6);
        case 7: SPARSP_F32_LAUNCH(7);
        case 8: SPARSP_F32_LAUNCH(8);
    }
#undef SPARSP_F32_LAUNCH
    return hipErrorInvalidValue;
}

}  // namespace sparsp
