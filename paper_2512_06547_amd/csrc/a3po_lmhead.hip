// Token log-probs straight from hidden states and the LM-head weight: z = h W^T is produced tile by tile on the
// matrix cores (a3po_gemm.hip, with the vocabulary on the row side and the tokens on the column side of the
// tile) and folded into a running (max, sum) per token as each tile leaves the accumulators, so the [T, V]
// logits never exist in memory.  A small kernel then merges the partials of the workgroups that shared a
// token, adds the chosen logit (a separate dot product) and writes log pi.
#include "a3po_common.h"
#include "a3po_launch.h"
#include "a3po_direct.h"
#include <type_traits>

namespace a3po {

// ---- few tokens -------------------------------------------------------------------------------------------------
// Up to 256 tokens the projection is bound by reading the weight (at 256 by the products as much), and the contraction
// kernel, whose ring holds three stages of 16 KiB of it ahead, reads 3.6 TB/s.  Here the weight does not pass through LDS at
// all: a wavefront owns two blocks of 16 vocabulary entries and loads their rows straight into MFMA operands (lane l: row
// l & 15, 16 bytes at quarter l >> 4; the two loads of a row block and chunk complete each 128-byte line), four chunks of 64
// hidden elements ahead: 96 to 128 KiB in flight per compute unit.  The workgroups start at different chunks: all of them at
// the same offset of rows 8 KiB apart would meet on a few memory channels (16 tokens x 4,096 x 151,936: 309 us so, 247 us
// apart, before the last round was spread; non-temporal loads, which let go of a line after its first half, are slower).  The
// hidden rows, which all wavefronts share, come through a ring of four chunks in LDS by direct loads; 16-byte piece p of row r
// sits at piece p ^ ((r >> 1) & 7), so that 16 consecutive rows of one piece fall into distinct banks.  32 rows per wavefront,
// because every operand read from LDS then feeds two MFMAs (with 16 rows and 256 tokens LDS would be the bound); kAhead of
// those reads are on the way (two, the compiler's choice: 376 instead of 340 us for 200 tokens).  One workgroup per compute
// unit, static tiles of 256 vocabulary entries.
//
// NB: 16-token column blocks.  H is a multiple of 256 (the loop is unrolled by the ring).  Operations in flight are
// counted by hand as in the contraction kernel: per chunk NB / 4 direct loads, then 4 operand loads (2 in the loop with one
// row block, whose first chunks thus wait for a little more than they need), in this order (held to in the source by
// in_order; tests/test_schedule.py reads it off the compiled kernel).
//
// A tile is 16 row blocks of 16, two per wavefront, but the tiles of the last round have only as many (last_blocks) as spread
// its rows over all compute units (FewTiles, which keeps to whole tiles where that gains nothing): a wavefront without a first or second block multiplies the tile's first row,
// whose lines all its lanes share, and leaves the products out of the fold.  A compute unit streams the weight at its own pace
// whatever the others do, so a third round of 82 whole tiles took as long as the two full ones before it (16 tokens x 4,096 x
// 151,936 247 us, now 220; x 2,048 x 32,000, 125 tiles on 256 units, 39 and 30; reading the rows of another block instead of
// one row gains nothing: lines that two loads ask for at a time are fetched twice).  From 129 tokens on the products count
// too: where no wavefront has a second block, the last round is a loop without it (192 tokens x 4,096 x 151,936 310 -> 286
// us, 256: 345 -> 329; a branch inside the one loop spills the accumulators).
constexpr int kFewThreads = kFewWaves * kWave;
constexpr int kFewRing = 4;
constexpr int kAhead = 4;
constexpr int kFewMaxTokens = 256;
template <int NB> constexpr int kFewLdsBytes = kFewRing * NB * 16 * 128 + kFewWaves * NB * 16 * (int)sizeof(float2);

template <int NB>
__global__ __launch_bounds__(kFewThreads) void lmhead_few_tokens_kernel(const uint16_t *W,
                                                                        const uint16_t *__restrict__ h, int T, int H,
                                                                        int V, int nfull, int ntiles, int last_blocks,
                                                                        float2 *__restrict__ partial)
{
    constexpr int kSlot = NB * 16 * 128;  // bytes of one chunk of the hidden rows
    constexpr int kDma = NB / 4;          // direct loads per wavefront and chunk
    static_assert(NB % 4 == 0, "the loads of a chunk are dealt evenly");
    extern __shared__ __align__(16) char lds[];
    float2 *red = reinterpret_cast<float2 *>(lds + kFewRing * kSlot);  // [kFewWaves][NB * 16]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nch = H / 64;
    const int64_t row_bytes = (int64_t)H * 2;
    const int rot = (int)(blockIdx.x % (unsigned)nch);
    auto chunk_at = [&](int i) { return i + rot < nch ? i + rot : i + rot - nch; };  // the i-th chunk this workgroup takes
    float2 *my_red = red + wave * (NB * 16);
    for (int c = lane; c < NB * 16; c += kWave) my_red[c] = make_float2(kNegFloor, 0.0f);

    // hidden rows: load i of a chunk covers rows 8 i .. 8 i + 7, this wavefront's are i = wave * kDma + j
    const __amdgpu_buffer_rsrc_t hbuf = dma_buffer(h, (uint32_t)(T * row_bytes));  // (at most 256 rows of 2 MiB)
    uint32_t hoff[kDma];
#pragma unroll
    for (int j = 0; j < kDma; ++j) {
        const int r = (wave * kDma + j) * 8 + (lane >> 3);
        hoff[j] = (uint32_t)(min(r, T - 1) * row_bytes) + (uint32_t)(((lane & 7) ^ ((r >> 1) & 7)) * 16);
    }
    auto load_hidden = [&](int slot, int chunk) {
#pragma unroll
        for (int j = 0; j < kDma; ++j) dma16(hbuf, hoff[j], (uint32_t)chunk_at(chunk) * 128u, lds + slot * kSlot + (wave * kDma + j) * 1024);
    };
    // weight rows of a tile: this lane's two row blocks (rows past the vocabulary are clamped and masked below)
    const char *wcur[2], *wnext[2];
    auto base_of = [&](int tile) { return tile < nfull ? tile * kFewRows : nfull * kFewRows + (tile - nfull) * last_blocks * 16; };
    auto has = [&](int tile, int r) { return tile < nfull || r * kFewWaves + wave < last_blocks; };
    auto rows_of = [&](int tile, const char **p) {
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int v = has(tile, r) ? base_of(tile) + (r * kFewWaves + wave) * 16 + (lane & 15) : base_of(tile);
            p[r] = reinterpret_cast<const char *>(W) + min(v, V - 1) * row_bytes + (lane >> 4) * 16;
        }
    };
    bf16x8_t a[kFewRing][2][2];  // [chunk mod ring][row block][half of the chunk]
    auto load_weight = [&](int j, const char *const *p, int i, int rows = 2) {
        const int chunk = chunk_at(i);
#pragma unroll
        for (int r = 0; r < rows; ++r)
#pragma unroll
            for (int k = 0; k < 2; ++k)
                a[j][r][k] = __builtin_bit_cast(
                    bf16x8_t, *reinterpret_cast<const u32x4_t *>(p[r] + chunk * 128 + k * 64));
    };
    // a hidden-row operand: row lane & 15 of block b, piece 4 k + (lane >> 4)
    const uint32_t brow = (uint32_t)(lane & 15) * 128u, bswz = (uint32_t)((lane >> 1) & 7);
    const uint32_t bpiece[2] = {brow + (((uint32_t)(lane >> 4)) ^ bswz) * 16u, brow + ((4u + (uint32_t)(lane >> 4)) ^ bswz) * 16u};

    // Keeps the two kinds of loads in the order that is counted on: the compiler moves no load across the memory clobber
    // (W is no __restrict__ pointer, through which it would) and no instruction across the scheduling barrier.
    auto in_order = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };

    int tile = blockIdx.x;  // (the grid has no more workgroups than there are tiles)
    rows_of(tile, wcur);
#pragma unroll
    for (int j = 0; j < kFewRing; ++j) {
        load_weight(j, wcur, j);
        in_order();
        if (j < kFewRing - 1) load_hidden(j, j);
        in_order();
    }
    // one tile, of whose row blocks this wavefront has the first `rows`
    auto take_tile = [&](auto rows) __attribute__((always_inline)) {
        constexpr int kRows = decltype(rows)::value;
        rows_of(tile + (int)gridDim.x < ntiles ? tile + (int)gridDim.x : tile, wnext);  // (past the end: read again, unused)
        f32x4_t acc[kRows][NB];
#pragma unroll
        for (int r = 0; r < kRows; ++r)
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[r][b][i] = 0.0f;
#pragma unroll 1
        for (int c = 0; c < nch; c += kFewRing) {
            const bool last = c + kFewRing >= nch;
#pragma unroll
            for (int j = 0; j < kFewRing; ++j) {
                __builtin_amdgcn_sched_barrier(0);
                // this chunk's hidden rows have landed (own loads: everything issued after them may still fly) and the
                // reads of the chunk before are done: meet, then refill the slot of the chunk before
                __builtin_amdgcn_s_waitcnt(waitcnt_imm(3 * 2 * kRows + 2 * kDma, 0));
                __builtin_amdgcn_s_barrier();
                __builtin_amdgcn_sched_barrier(0);
                const int ahead = c + j + kFewRing - 1;
                load_hidden((j + kFewRing - 1) % kFewRing, ahead < nch ? ahead : ahead - nch);
                in_order();
                const char *stage = lds + j * kSlot;
                // 2 NB operands of hidden rows, kAhead of them on the way while one is used
                bf16x8_t fb[kAhead + 1];
                auto read = [&](int i) {
                    fb[i % (kAhead + 1)] = *reinterpret_cast<const bf16x8_t *>(stage + (i % NB) * 2048 + bpiece[i / NB]);
                };
#pragma unroll
                for (int i = 0; i < kAhead; ++i) read(i);
#pragma unroll
                for (int i = 0; i < 2 * NB; ++i) {
                    if (i + kAhead < 2 * NB) read(i + kAhead);
#pragma unroll
                    for (int r = 0; r < kRows; ++r)
                        acc[r][i % NB] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[j][r][i / NB], fb[i % (kAhead + 1)],
                                                                                 acc[r][i % NB], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
                in_order();
                load_weight(j, last ? wnext : wcur, last ? c + j + kFewRing - nch : c + j + kFewRing, kRows);
                in_order();
            }
        }
        // fold the tile: accumulator (r, b, i) is entry 4 (lane >> 4) + i of this wavefront's row block r, token b 16 + (lane & 15)
        int left[kRows];
#pragma unroll
        for (int r = 0; r < kRows; ++r) left[r] = has(tile, r) ? V - base_of(tile) - (r * kFewWaves + wave) * 16 - 4 * (lane >> 4) : 0;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            float f[4 * kRows];
#pragma unroll
            for (int r = 0; r < kRows; ++r)
#pragma unroll
                for (int i = 0; i < 4; ++i) f[r * 4 + i] = i < left[r] ? acc[r][b][i] : -INFINITY;
            MaxSum mine = {kNegFloor, 0.0f};
            fold<4 * kRows>(mine, f);
#pragma unroll
            for (int off = 16; off <= 32; off <<= 1) {
                const MaxSum other = {__shfl_xor(mine.m, off, kWave), __shfl_xor(mine.s, off, kWave)};
                mine = combine(mine, other);
            }
            if (lane < 16) {  // (this wavefront's own row of red)
                const f32x2_t q = lds_get<f32x2_t>(my_red + b * 16 + lane);
                mine = combine(MaxSum{q[0], q[1]}, mine);
                lds_put(my_red + b * 16 + lane, f32x2_t{mine.m, mine.s});
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int r = 0; r < 2; ++r) wcur[r] = wnext[r];
        tile += (int)gridDim.x;
    };
    // (no test before the first tile: the loads above would be moved behind it)
    const int nloop = NB >= 12 && nfull > 0 && last_blocks <= kFewWaves ? nfull : ntiles;
    do {
        take_tile(std::integral_constant<int, 2>());
    } while (tile < nloop);
    if constexpr (NB >= 12)
        if (tile < ntiles) take_tile(std::integral_constant<int, 1>());
    __syncthreads();  // (also drains the loads past the last tile)
    if (tid < NB * 16 && tid < T) {
        MaxSum tot = {kNegFloor, 0.0f};
        for (int w = 0; w < kFewWaves; ++w) {
            const float2 q = red[w * (NB * 16) + tid];
            tot = combine(tot, MaxSum{q.x, q.y});
        }
        partial[(int64_t)blockIdx.x * T + tid] = make_float2(tot.m, tot.s);
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));
}

// z[t, y_t] = h[t, :] . W[y_t, :] in fp32, one wavefront per token; then
// lse_t from the partials of the workgroups that swept this token and log pi = z_y - lse.
// Bound by latency (two rows and a strided column of partials per wavefront): the dot product keeps four pairs of
// 16-byte loads in flight, and the partials are spread over the lanes and merged by the wavefront (200 tokens x 4,096:
// 24 us with one load pair at a time and one lane walking the partials).
__global__ __launch_bounds__(256) void lmhead_finish_kernel(const uint16_t *__restrict__ W,
                                                            const uint16_t *__restrict__ h, int64_t T, int64_t H,
                                                            int64_t V, const int32_t *__restrict__ chosen,
                                                            const float2 *__restrict__ partial, int nxcd, int per_xcd,
                                                            GemmCut host_cut, int64_t room, int slots, float *logp, float *lse_out, DynCount count)
{
    const int lane = threadIdx.x & 63;
    const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int64_t N = dyn_extent(count, T);
    if (t >= N) return;
    const int32_t y = chosen[t];
    const bool ok = y >= 0 && (int64_t)y < V;
    MaxSum tot = {kNegFloor, 0.0f};
    // (slots > 0: that many partials, all of them written)
    for (int p = lane; p < slots; p += kWave) {
        const float2 q = partial[(int64_t)p * N + t];
        tot = combine(tot, MaxSum{q.x, q.y});
    }
    if (slots == 0) {
        // slot (xcd, m) holds a partial of this token if that XCD's range of pairs met the token's column group in a round
        // that has a tile for row m of the block (GemmCut)
        const GemmCut cut = count.n ? gemm_cut(V, N, nxcd, per_xcd, room) : host_cut;
        const int tile = (int)(t / kGemmTile);
        const int64_t c0 = min((int64_t)cut.tiles0 * kGemmTile, N);
        const bool two = tile >= cut.tiles0;
        const int ml = two ? cut.part[1].ml : cut.part[0].ml, rounds = two ? cut.part[1].rounds : cut.part[0].rounds;
        const int64_t g0 = two ? cut.pairs0 + (int64_t)((tile - cut.tiles0) / cut.part[1].ncol) * rounds : (int64_t)(tile / cut.part[0].ncol) * rounds;
        const float2 *mine = two ? partial + (int64_t)nxcd * cut.part[0].ml * c0 + (t - c0) : partial + t;
        const int64_t width = two ? N - c0 : c0;
        for (int p = lane; p < nxcd * ml; p += kWave) {
            const int xcd = p / ml, m = p % ml;
            const int64_t lo = max((int64_t)xcd * cut.pairs / nxcd, g0), hi = min((int64_t)(xcd + 1) * cut.pairs / nxcd, g0 + rounds);
            if (lo < hi && (lo - g0) * ml + m < cut.part[0].mtiles) {
                const float2 q = mine[(int64_t)p * width];
                tot = combine(tot, MaxSum{q.x, q.y});
            }
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
                                    float *lse, hipStream_t s, int64_t room, DynCount count, int slots)
{
    const unsigned grid = (unsigned)((T + 3) / 4);
    const GemmGrid gg = gemm_grid();
    // (the kernel searches the cut itself where the number of tokens is on the device, and needs none for `slots` partials)
    const GemmCut cut = slots > 0 || count.n ? GemmCut() : gemm_cut(V, T, gg.nxcd, gg.per_xcd, room);
    hipLaunchKernelGGL(lmhead_finish_kernel, dim3(grid), dim3(256), 0, s, reinterpret_cast<const uint16_t *>(weight),
                       reinterpret_cast<const uint16_t *>(hidden), T, H, V, chosen, partial, gg.nxcd, gg.per_xcd, cut, room, slots,
                       logp, lse, count);
    return hipGetLastError();
}

template <int NB>
static hipError_t launch_few_tokens(const void *hidden, const void *weight, int64_t T, int64_t H, int64_t V, float2 *partial,
                                    const FewTiles &ft, hipStream_t s)
{
    static LdsLimitState lds_limit;
    auto *kernel = lmhead_few_tokens_kernel<NB>;
    const hipError_t e = ensure_lds_limit(reinterpret_cast<const void *>(kernel), kFewLdsBytes<NB>, lds_limit);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(ft.slots), dim3(kFewThreads), kFewLdsBytes<NB>, s, reinterpret_cast<const uint16_t *>(weight),
                       reinterpret_cast<const uint16_t *>(hidden), (int)T, (int)H, (int)V, ft.nfull, ft.ntiles, ft.last_blocks,
                       partial);
    return hipGetLastError();
}

hipError_t launch_fused_lmhead_logprob(const void *hidden, const void *weight, int64_t T, int64_t H, int64_t V,
                                       const int32_t *chosen, float *logp, float *lse, void *workspace, hipStream_t s)
{
    if (T == 0) return hipSuccess;
    float2 *partial = reinterpret_cast<float2 *>(workspace);
    // Few tokens: the kernel for them up to 192; from 193 to 256 where its tiles occupy most compute units (every tile
    // reads the T x H x 2 bytes of hidden rows, which at 256 tokens weigh as much as its 256 x H x 2 bytes of weight).
    // Contraction kernel / this one, us:
    // 16 / 128 / 192 / 200 tokens x 4,096 x 151,936 347 / 334 / 346 / 346 and 220 / 255 / 286 / 318; 192 x 4,096 x 16,000 / 40,000
    // 79 / 113 and 70 / 94; small vocabularies, 129 x 256 x 2,000 / 16,000 17.6 / 17.1 and 15.1 / 16.3, 192 x 1,024 x 1,000 /
    // 24,000 29.3 / 30.2 and 24.4 / 27.5, 160 x 4,096 x 500 / 12,000 77.1 / 78.1 and 64.9 / 68.8; 250 x 2,048 x 128,256 156 and
    // 139, 250 x 1,536 x 50,264 (197 tiles) 58 and 57, 200 x 2,048 x 32,000 (125 tiles) 47 and 56.
    const GemmGrid gg = gemm_grid();
    const int64_t tiles = (V + kFewRows - 1) / kFewRows, cus = (int64_t)gg.nxcd * gg.per_xcd;
    const bool few = T <= 192 || (T <= kFewMaxTokens && tiles >= cus * 3 / 4);
    if (few && H % 256 == 0 && V <= 0x7FFFFFFF - 256 * kFewRows) {
        const FewTiles ft = few_tiles_of(T, V, cus);  // at most 256 slots: gemm_partial_entries(T) is 256 T here
        const hipError_t e = T <= 64    ? launch_few_tokens<4>(hidden, weight, T, H, V, partial, ft, s)
                             : T <= 128 ? launch_few_tokens<8>(hidden, weight, T, H, V, partial, ft, s)
                             : T <= 192 ? launch_few_tokens<12>(hidden, weight, T, H, V, partial, ft, s)
                                        : launch_few_tokens<16>(hidden, weight, T, H, V, partial, ft, s);
        if (e != hipSuccess) return e;
        return launch_lmhead_lse_finish(hidden, weight, T, H, V, chosen, partial, logp, lse, s, 0, DynCount(), ft.slots);
    }
    GemmArgs g = {};
    g.A = reinterpret_cast<const uint16_t *>(weight);
    g.lda = H;
    g.B = reinterpret_cast<const uint16_t *>(hidden);
    g.ldb = H;
    g.M = V;
    g.N = T;
    g.K = H;
    g.partial = partial;
    g.room = (int64_t)gemm_partial_entries(T);
    hipError_t e = launch_gemm(g, kGemmLse, s);
    if (e != hipSuccess) return e;
    return launch_lmhead_lse_finish(hidden, weight, T, H, V, chosen, g.partial, logp, lse, s, g.room);
}

}  // namespace a3po
