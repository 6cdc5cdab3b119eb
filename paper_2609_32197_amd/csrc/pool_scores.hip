// Step 1: pooled query/key tiles and block scores (Section 4.2).
//
// pool_kernel: one workgroup per (head, block) streams the block's rows from
// HBM with 16-byte non-temporal loads (every lane of a row group reads one
// 16-byte chunk, so a row group covers a whole token row: fully coalesced),
// accumulates float32 column sums in registers, reduces the row groups
// through LDS in a fixed order and divides by the block's valid token count.
// Q's local blocks and all of K's blocks go through one launch. The step is
// HBM-bound.
//
// score_kernel: per head, scores = pooled_q · pooled_k^T · d^-1/2 in float32 on
// the matrix cores (v_mfma_f32_16x16x4_f32): a 64x64 output tile per workgroup,
// 32x32 per wave, d staged through LDS in slices of 32. About 1 GFLOP and 30 MB
// at the largest workload, so latency bounds it more than the 8 us of its
// products: 40 heads x 147 x 591 blocks, d = 128 36.6 us with float32 FMAs on
// transposed LDS tiles, 25.6 with slices of 64 (34 KB of LDS: a second round of
// workgroups), 22.2 as it is; 48 x 139 x 278, d = 64 18.1 and 11.0 us.
#include "sparsp_internal.h"

namespace sparsp {
namespace {

constexpr int kPoolThreads = 256;

template <bool BF16>
__global__ __launch_bounds__(kPoolThreads) void pool_kernel(
    const void* __restrict__ Q, const void* __restrict__ K, float* __restrict__ pooled_q,
    float* __restrict__ pooled_k, int H, int L, int d, int block, int i0, int nq, int n) {
    // Elements per 16-byte chunk.
    constexpr int VEC = BF16 ? 8 : 4;
    __shared__ float part[kPoolThreads * VEC];

    const int h = blockIdx.y;
    int t = blockIdx.x;  // [0, nq) -> Q block i0+t ; [nq, nq+n) -> K block t-nq
    const bool is_q = t < nq;
    const int blk = is_q ? i0 + t : t - nq;
    const char* src = static_cast<const char*>(is_q ? Q : K);
    float* dst = is_q ? pooled_q + (int64_t(h) * nq + t) * d
                      : pooled_k + (int64_t(h) * n + (t - nq)) * d;

    const int tok0 = blk * block;
    const int cnt = min(block, L - tok0);
    const int chunks = d / VEC;                 // chunks per token row
    const int groups = kPoolThreads / chunks;   // row groups; >= 4 because d <= 256
    const int tid = threadIdx.x;
    const int ch = tid % chunks;
    const int rg = tid / chunks;

    float acc[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] = 0.f;

    if (rg < groups) {
        const int64_t esize = BF16 ? 2 : 4;
        const char* base = src + ((int64_t(h) * L + tok0) * d + int64_t(ch) * VEC) * esize;
        const int64_t row_bytes = int64_t(d) * esize;
        int r = rg;
        // Four rows in flight per iteration. Non-temporal loads: Q and K are
        // read once here, and with the hint a cold read runs about a quarter
        // faster.
        for (; r + 3 * groups < cnt; r += 4 * groups) {
            uint4 x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] = load_nt(base + int64_t(r + u * groups) * row_bytes);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t w[4] = {x[u].x, x[u].y, x[u].z, x[u].w};
                if constexpr (BF16) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        acc[2 * v] += bf16_bits_to_f32(w[v] & 0xffffu);
                        acc[2 * v + 1] += bf16_bits_to_f32(w[v] >> 16);
                    }
                } else {
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[v] += __uint_as_float(w[v]);
                }
            }
        }
        for (; r < cnt; r += groups) {
            const uint4 x = load_nt(base + int64_t(r) * row_bytes);
            const uint32_t w[4] = {x.x, x.y, x.z, x.w};
            if constexpr (BF16) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    acc[2 * v] += bf16_bits_to_f32(w[v] & 0xffffu);
                    acc[2 * v + 1] += bf16_bits_to_f32(w[v] >> 16);
                }
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[v] += __uint_as_float(w[v]);
            }
        }
    }
    // part[rg][ch*VEC + v]; threads past the last full row group hold nothing.
    if (rg < groups) {
#pragma unroll
        for (int v = 0; v < VEC; ++v) part[rg * d + ch * VEC + v] = acc[v];
    }
    __syncthreads();
    for (int c = tid; c < d; c += kPoolThreads) {
        float s = 0.f;
        for (int q = 0; q < groups; ++q) s += part[q * d + c];
        dst[c] = s / float(cnt);
    }
}

constexpr int kTile = 64;   // output tile edge
constexpr int kSlice = 32;  // d slice staged per step
constexpr int kPitch = kSlice + 4;  // floats per LDS row: 16 rows start on 16 different banks of 16 bytes

typedef float floatx4 __attribute__((ext_vector_type(4)));

// VEC: the pooled tiles are 16-byte aligned (their rows then are too, d being a
// multiple of 4).
template <bool VEC>
__device__ __forceinline__ floatx4 load4(const float* p) {
    if constexpr (VEC) return *reinterpret_cast<const floatx4*>(p);
    return floatx4{p[0], p[1], p[2], p[3]};
}

template <bool VEC>
__global__ __launch_bounds__(256) void score_kernel(const float* __restrict__ pq,
                                                     const float* __restrict__ pk,
                                                     float* __restrict__ scores, int nq, int n,
                                                     int d, float scale) {
    __shared__ __attribute__((aligned(16))) float As[kTile * kPitch];
    __shared__ __attribute__((aligned(16))) float Bs[kTile * kPitch];
    const int h = blockIdx.z;
    const int row0 = blockIdx.y * kTile;  // query blocks
    const int col0 = blockIdx.x * kTile;  // key blocks
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int qi = lane & 15, g = lane >> 4;
    const int wr = 32 * (wave >> 1), wc = 32 * (wave & 1);  // this wave's 32x32 outputs
    const float* A = pq + int64_t(h) * nq * d;
    const float* B = pk + int64_t(h) * n * d;

    // A slice is 64 rows of 8 float4 per operand, two of each per thread; the
    // next slice is read while this one is multiplied.
    floatx4 xa[2], xb[2];
    const int r4 = tid >> 3, c4 = (tid & 7) * 4;
    auto fetch = [&](int k0) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int ra = row0 + r4 + 32 * i, rb = col0 + r4 + 32 * i, k = k0 + c4;
            xa[i] = (ra < nq && k < d) ? load4<VEC>(A + int64_t(ra) * d + k) : floatx4{};
            xb[i] = (rb < n && k < d) ? load4<VEC>(B + int64_t(rb) * d + k) : floatx4{};
        }
    };
    floatx4 acc[2][2] = {};
    fetch(0);
    for (int k0 = 0; k0 < d; k0 += kSlice) {
        if (k0 > 0) __syncthreads();  // every wave is done with the slice before
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            *reinterpret_cast<floatx4*>(&As[(r4 + 32 * i) * kPitch + c4]) = xa[i];
            *reinterpret_cast<floatx4*>(&Bs[(r4 + 32 * i) * kPitch + c4]) = xb[i];
        }
        __syncthreads();
        if (k0 + kSlice < d) fetch(k0 + kSlice);
        // Lane group g supplies elements 16 c + 4 g + u of both operands in
        // product u of chunk c.
#pragma unroll
        for (int c = 0; c < kSlice / 16; ++c) {
            floatx4 a[2], b[2];
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                a[x] = *reinterpret_cast<const floatx4*>(&As[(wr + 16 * x + qi) * kPitch + 16 * c + 4 * g]);
                b[x] = *reinterpret_cast<const floatx4*>(&Bs[(wc + 16 * x + qi) * kPitch + 16 * c + 4 * g]);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int x = 0; x < 2; ++x)
#pragma unroll
                    for (int y = 0; y < 2; ++y)
                        acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[x][u], b[y][u], acc[x][y],
                                                                         0, 0, 0);
        }
    }
    // The lane holds rows 4 g .. +3 of column qi of each 16x16 tile.
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = row0 + wr + 16 * x + 4 * g + r;
            if (i >= nq) continue;
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                const int j = col0 + wc + 16 * y + qi;
                if (j < n) scores[(int64_t(h) * nq + i) * n + j] = acc[x][y][r] * scale;
            }
        }
}

}  // namespace

hipError_t launch_pool_scores(const Geom& g, const void* Q, const void* K, float* pooled_q,
                              float* pooled_k, float* scores, hipStream_t s) {
    (void)hipGetLastError();
    dim3 pgrid(g.nq + g.n, g.H);
    if (g.bf16)
        pool_kernel<true><<<pgrid, kPoolThreads, 0, s>>>(Q, K, pooled_q, pooled_k, g.H, g.L, g.d,
                                                         g.block, g.i0, g.nq, g.n);
    else
        pool_kernel<false><<<pgrid, kPoolThreads, 0, s>>>(Q, K, pooled_q, pooled_k, g.H, g.L, g.d,
                                                          g.block, g.i0, g.nq, g.n);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    dim3 sgrid((g.n + kTile - 1) / kTile, (g.nq + kTile - 1) / kTile, g.H);
    const float scale = 1.0f / sqrtf(float(g.d));
    const bool vec = ((reinterpret_cast<uintptr_t>(pooled_q) | reinterpret_cast<uintptr_t>(pooled_k)) & 15) == 0;
    auto* score = vec ? score_kernel<true> : score_kernel<false>;
    score<<<sgrid, 256, 0, s>>>(pooled_q, pooled_k, scores, g.nq, g.n, g.d, scale);
    return hipGetLastError();
}

}  // namespace sparsp
