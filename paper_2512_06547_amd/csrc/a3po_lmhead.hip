// Token log-probs straight from hidden states and the LM-head weight: z = h W^T is produced tile by tile on the
// matrix cores (a3po_gemm.hip, with the vocabulary on the row side and the tokens on the column side of the
// tile) and folded into a running (max, sum) per token as each tile leaves the accumulators, so the [T, V]
// logits never exist in memory.  A small kernel then merges the partials of the workgroups that shared a
// token, adds the chosen logit (a separate dot product) and writes log pi.
#include "a3po_common.h"
#include "a3po_launch.h"

namespace a3po {

// z[t, y_t] = h[t, :] . W[y_t, :] in fp32, one wavefront per token; then
// lse_t from the partials of the workgroups that swept this token and log pi = z_y - lse.
// Bound by latency (two rows and a strided column of partials per wavefront): the dot product keeps four pairs of
// 16-byte loads in flight, and the partials are spread over the lanes and merged by the wavefront (200 tokens x 4,096:
// 24 us with one load pair at a time and one lane walking the partials).
__global__ __launch_bounds__(256) void lmhead_finish_kernel(const uint16_t *__restrict__ W,
                                                            const uint16_t *__restrict__ h, int64_t T, int64_t H,
                                                            int64_t V, const int32_t *__restrict__ chosen,
                                                            const float2 *__restrict__ partial, int nxcd, int per_xcd,
                                                            float *logp, float *lse_out, DynCount count)
{
    const int lane = threadIdx.x & 63;
    const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int64_t N = dyn_extent(count, T);
    if (t >= N) return;
    const int32_t y = chosen[t];
    const bool ok = y >= 0 && (int64_t)y < V;
    // slot (xcd, m) holds a partial of this token if that XCD's range of pairs met the token's column group in a round
    // that has a tile for row m of the block (GemmShape)
    const GemmShape shp = gemm_shape(V, N, nxcd, per_xcd);
    const int64_t pairs = (int64_t)shp.groups * shp.rounds, g0 = (t / kGemmTile / shp.ncol) * shp.rounds;
    MaxSum tot = {kNegFloor, 0.0f};
    for (int p = lane; p < nxcd * shp.ml; p += kWave) {
        const int xcd = p / shp.ml, m = p % shp.ml;
        const int64_t lo = max((int64_t)xcd * pairs / nxcd, g0), hi = min((int64_t)(xcd + 1) * pairs / nxcd, g0 + shp.rounds);
        if (lo < hi && (lo - g0) * shp.ml + m < shp.mtiles) {
            const float2 q = partial[(int64_t)p * N + t];
            tot = combine(tot, MaxSum{q.x, q.y});
        }
    }
    float dot = 0.0f;
    if (ok) {
        const uint16_t *hr = h + t * H, *wr = W + (int64_t)y * H;
        constexpr int kUnroll = 4;
        for (int64_t k0 = (int64_t)lane * 8; k0 < H; k0 += kUnroll * 64 * 8) {
            uint4 a[kUnroll], b[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const int64_t k = k0 + u * 64 * 8;
                a[u] = b[u] = make_uint4(0u, 0u, 0u, 0u);
                if (k < H) {
                    a[u] = *reinterpret_cast<const uint4 *>(hr + k);
                    b[u] = *reinterpret_cast<const uint4 *>(wr + k);
                }
            }
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                float fa[8], fb[8];
                unpack<Bf16>(a[u], fa);
                unpack<Bf16>(b[u], fb);
#pragma unroll
                for (int e = 0; e < 8; ++e) dot = fmaf(fa[e], fb[e], dot);
            }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) dot += __shfl_xor(dot, off, kWave);
    }
    tot = wave_reduce(tot);
    if (lane == 0) {
        const float log_s = logf(tot.s);
        if (lse_out) lse_out[t] = tot.m + log_s;
        logp[t] = ok ? (dot - tot.m) - log_s : 0.0f;
    }
}

size_t lmhead_workspace_bytes(int64_t T)
{
    const size_t t = (size_t)(T > 0 ? T : 0);
    return ((gemm_partial_entries((int64_t)t) * sizeof(float2) + 255) / 256) * 256 + 256;
}

hipError_t launch_lmhead_lse_finish(const void *hidden, const void *weight, int64_t T, int64_t H, int64_t V,
                                    const int32_t *chosen, const float2 *partial, float *logp,
                                    float *lse, hipStream_t s, DynCount count)
{
    const unsigned grid = (unsigned)((T + 3) / 4);
    const GemmGrid gg = gemm_grid();
    hipLaunchKernelGGL(lmhead_finish_kernel, dim3(grid), dim3(256), 0, s, reinterpret_cast<const uint16_t *>(weight),
                       reinterpret_cast<const uint16_t *>(hidden), T, H, V, chosen, partial, gg.nxcd, gg.per_xcd, logp,
                       lse, count);
    return hipGetLastError();
}

hipError_t launch_fused_lmhead_logprob(const void *hidden, const void *weight, int64_t T, int64_t H, int64_t V,
                                       const int32_t *chosen, float *logp, float *lse, void *workspace, hipStream_t s)
{
    if (T == 0) return hipSuccess;
    GemmArgs g = {};
    g.A = reinterpret_cast<const uint16_t *>(weight);
    g.lda = H;
    g.B = reinterpret_cast<const uint16_t *>(hidden);
    g.ldb = H;
    g.M = V;
    g.N = T;
    g.K = H;
    g.partial = reinterpret_cast<float2 *>(workspace);
    hipError_t e = launch_gemm(g, kGemmLse, s);
    if (e != hipSuccess) return e;
    return launch_lmhead_lse_finish(hidden, weight, T, H, V, chosen, g.partial, logp, lse, s);
}

}  // namespace a3po
