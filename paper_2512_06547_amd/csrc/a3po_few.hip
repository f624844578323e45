// Loss forward + backward of a short batch: every row is cut into parts, one workgroup each.
//
// With a workgroup per row (a3po_rows.hip) a batch of fewer rows than compute units leaves most of the chip idle, and its
// time is that of one unit reading and writing one row (64 of bfloat16 x 151,936: 29.3 us a pass, 22.0 so), behind a kernel that
// packs the records and before one that adds up the loss.  Here all units share the rows, in two launches:
//   1. (max, sum[, sum of exp(z - m) z]) of each part, while one more workgroup packs the records and writes the header;
//   2. every workgroup merges its row's partials (each in the same order, so all agree to the bit), works out the token's
//      terms and writes its part of the gradient; one more does the same for every token and writes the per-token
//      outputs, the loss and the statistics.
// Bound by latency (launches, one round of loads each) up to some 64 rows, then by reading the logits twice, the second time
// from the caches.  Log-probs, loss, statistics and gradient are those of the row kernel up to the order of the sums.
// A row's parts are whole 128-byte lines of the gradient, so that no store straddles one; the elements before its first line
// go to the first part, those behind its last whole vector to the last.  Logits and gradient may sit at any element
// alignment.  The second launch reads no caller's array that it or another workgroup writes: a part reads its own logits
// before it overwrites them (the gradient may take the logits' place), the chosen logit travels with the partials.
#include "a3po_common.h"
#include "a3po_launch.h"
#include "a3po_row_plan.h"
#include "a3po_tokens.h"

namespace a3po {

constexpr int kFewUnroll = 4;  // 16-byte vectors in flight per thread

// this workgroup's part of a row: elements before the first line, vectors [first, last) of the body, elements behind it
struct FewPart {
    int head, first, last, tail0, tail;
};

template <typename DT>
__device__ __forceinline__ FewPart few_part(const char *out_row, int V, int part, int parts)
{
    const uint32_t to_line = (0u - (uint32_t)reinterpret_cast<uintptr_t>(out_row)) & 127u;
    const int head = min(V, (int)(to_line / DT::kBytes)), nbody = (V - head) / DT::kPerVec;
    const int per = ((nbody + parts - 1) / parts + 7) / 8 * 8;
    FewPart p;
    p.head = head;
    p.first = min(nbody, part * per);
    p.last = min(nbody, p.first + per);
    p.tail0 = head + nbody * DT::kPerVec;
    p.tail = V - p.tail0;
    return p;
}

// the column of the single element this thread holds, or -1 (threads 0 .. 62 the head's, 64 .. 70 the tail's)
__device__ __forceinline__ int few_single(const FewPart &p, int part, int parts, int tid)
{
    if (part == 0 && tid < p.head) return tid;
    if (part == parts - 1 && tid >= kWave && tid - kWave < p.tail) return p.tail0 + tid - kWave;
    return -1;
}

// The reductions of a3po_common.h with the multiply-adds written out: the compiler chooses which product of a sum to fuse,
// and may choose differently with and without u, but asking for the entropy must not change the log-probs.
template <bool ENT>
__device__ __forceinline__ MaxSumU few_combine(MaxSumU a, MaxSumU b)
{
    MaxSumU o = {fmaxf(a.m, b.m), 0.0f, 0.0f};
    const float fa = exp2_hw((a.m - o.m) * kLog2e), fb = exp2_hw((b.m - o.m) * kLog2e);
    o.s = fmaf(a.s, fa, b.s * fb);
    if constexpr (ENT) o.u = fmaf(a.u, fa, b.u * fb);
    return o;
}

template <int N, bool ENT>
__device__ __forceinline__ void few_fold(MaxSumU &acc, const float *f)
{
    float m = acc.m;
#pragma unroll
    for (int e = 0; e < N; ++e) m = fmaxf(m, f[e]);
    const float scale = exp2_hw((acc.m - m) * kLog2e);
    if constexpr (ENT) acc.u *= scale;
#pragma unroll
    for (int e = 0; e < N; ++e) {
        const float ex = exp2_hw((f[e] - m) * kLog2e);
        acc.s = e == 0 ? fmaf(acc.s, scale, ex) : acc.s + ex;
        if constexpr (ENT) acc.u = fmaf(ex, finite_floor(f[e]), acc.u);
    }
    acc.m = m;
}

// A row's partials, (m, s, chosen logit (part 0's alone), u) each, in the order of the parts.
template <bool ENT>
__device__ __forceinline__ MaxSumU few_merge(const float4 *__restrict__ partial, int parts)
{
    MaxSumU t = {kNegFloor, 0.0f, 0.0f};
    for (int p = 0; p < parts; ++p) t.m = fmaxf(t.m, partial[p].x);
    for (int p = 0; p < parts; ++p) {
        const float f = exp2_hw((partial[p].x - t.m) * kLog2e);
        t.s = fmaf(partial[p].y, f, t.s);
        if constexpr (ENT) t.u = fmaf(partial[p].w, f, t.u);
    }
    return t;
}

template <typename DT, bool ENT, bool ANY>
__global__ __launch_bounds__(kTokThreads) void few_rows_partials_kernel(const LossArgs a, int parts)
{
    constexpr int EPV = DT::kPerVec;
    __shared__ MaxSumU red[kTokWaves];
    const int tid = threadIdx.x, row = (int)blockIdx.x / parts, part = (int)blockIdx.x % parts;
    if (row == (int)a.T) {
        const PrepPartial total = pack_records(a.chosen, a.mask, a.lb, a.prox_mode == A3PO_PROX_INTERP ? a.versions : nullptr, a.adv,
                                               a.prox_mode == A3PO_PROX_GIVEN ? a.prox_in : nullptr, 0, a.T, a.V, a.ws_records);
        if (tid == 0) write_header(total, a.denom_dev ? *a.denom_dev : a.denom, reinterpret_cast<WsHeader *>(a.ws_header));
        return;
    }
    const int32_t y = a.chosen[row];
    if (a.mask[row] == 0 || y < 0 || (int64_t)y >= a.V) return;
    const size_t at = (size_t)row * (size_t)a.ld * DT::kBytes;
    const char *in_row = reinterpret_cast<const char *>(a.z) + at;
    const FewPart p = few_part<DT>(reinterpret_cast<const char *>(a.dz) + at, (int)a.V, part, parts);
    const char *body = in_row + p.head * DT::kBytes;
    const uint32_t zy_bits = load_raw<DT>(in_row, y);
    const int single = few_single(p, part, parts, tid);
    const uint32_t single_bits = single >= 0 ? load_raw<DT>(in_row, single) : 0u;
    MaxSumU acc = {kNegFloor, 0.0f, 0.0f};
    for (int i0 = p.first; i0 < p.last; i0 += kFewUnroll * kTokThreads) {
        uint4 v[kFewUnroll];
#pragma unroll
        for (int u = 0; u < kFewUnroll; ++u) {
            const int i = i0 + u * kTokThreads + tid;
            if (i < p.last) v[u] = row_load<ANY, true>(body + (size_t)i * 16);
        }
#pragma unroll
        for (int u = 0; u < kFewUnroll; ++u) {
            if (i0 + u * kTokThreads + tid < p.last) {
                float f[EPV];
                unpack<DT>(v[u], f);
                few_fold<EPV, ENT>(acc, f);
            }
            __builtin_amdgcn_sched_barrier(0);  // one vector's temporaries at a time
        }
    }
    if (single >= 0) {
        float f[1] = {raw_to_float<DT>(single_bits)};
        few_fold<1, ENT>(acc, f);
    }
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        MaxSumU o = {__shfl_xor(acc.m, off, kWave), __shfl_xor(acc.s, off, kWave), 0.0f};
        if constexpr (ENT) o.u = __shfl_xor(acc.u, off, kWave);
        acc = few_combine<ENT>(acc, o);
    }
    if (tid % kWave == 0) red[tid / kWave] = acc;
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < kTokWaves; ++w) acc = few_combine<ENT>(acc, red[w]);
        reinterpret_cast<float4 *>(a.ws_scratch)[blockIdx.x] = make_float4(acc.m, acc.s, raw_to_float<DT>(zy_bits), acc.u);
    }
}

template <typename DT, bool ENT, bool ANY>
__global__ __launch_bounds__(kTokThreads) void few_rows_gradient_kernel(const LossArgs a, int parts)
{
    constexpr int EPV = DT::kPerVec;
    const WsHeader *hdr = reinterpret_cast<const WsHeader *>(a.ws_header);
    const float4 *partial = reinterpret_cast<const float4 *>(a.ws_scratch);
    const int tid = threadIdx.x, row = (int)blockIdx.x / parts, part = (int)blockIdx.x % parts;
    if (row == (int)a.T) {  // loss, statistics and per-token outputs: one token per thread
        FinishTotals mine = {0.0, 0.0, 0, 0, INFINITY, -INFINITY};
        if (tid < (int)a.T) {
            const TokenRecord rec = a.ws_records[tid];
            float lt = 0.0f, lp = 0.0f, iw = 0.0f, ent = 0.0f;
            bool clipped = false;
            if (rec.y >= 0) {
                const MaxSumU tot = few_merge<ENT>(partial + tid * parts, parts);
                const float log_s = logf(tot.s);
                lt = (partial[tid * parts].z - tot.m) - log_s;
                const TokenTerms tt = token_terms(lt, rec.lb, rec.ver, a.current_version, rec.A, a.clip_eps, hdr->inv_n, a.prox_mode);
                lp = tt.lp;
                iw = tt.iw;
                clipped = tt.clipped;
                if constexpr (ENT) ent = entropy_of(tot, tot.m + log_s);
                mine = {(double)tt.obj, (double)ent, clipped ? 1 : 0, tt.negative_staleness ? 1 : 0, fminf(INFINITY, iw),
                        fmaxf(-INFINITY, iw)};
            }
            a.logp_out[tid] = lt;
            if (a.prox_out) a.prox_out[tid] = lp;
            if constexpr (ENT) a.ent_out[tid] = ent;
            if (a.iw_out) a.iw_out[tid] = iw;
            if (a.clipped_out) a.clipped_out[tid] = clipped ? 1 : 0;
        }
        const FinishTotals tot = block_totals(mine);
        if (tid == 0) write_loss_and_stats(tot, ENT, hdr, a.loss_out, a.stats_out, a.accumulate);
        return;
    }
    const TokenRecord rec = a.ws_records[row];
    const size_t at = (size_t)row * (size_t)a.ld * DT::kBytes;
    const char *in_row = reinterpret_cast<const char *>(a.z) + at;
    char *out_row = reinterpret_cast<char *>(a.dz) + at;
    const FewPart p = few_part<DT>(out_row, (int)a.V, part, parts);
    const char *body = in_row + p.head * DT::kBytes;
    char *out = out_row + p.head * DT::kBytes;
    const int single = few_single(p, part, parts, tid);
    float g = 0.0f, row_max = 0.0f, nls2 = 0.0f, zy = 0.0f;
    if (rec.y >= 0) {
        const MaxSumU tot = few_merge<false>(partial + row * parts, parts);
        const float log_s = logf(tot.s);
        zy = partial[row * parts].z;
        row_max = tot.m;
        nls2 = -log_s * kLog2e;
        g = token_terms((zy - tot.m) - log_s, rec.lb, rec.ver, a.current_version, rec.A, a.clip_eps, hdr->inv_n, a.prox_mode).g;
    }
    if (g == 0.0f) {  // masked, invalid id, clipped, zero advantage or empty batch: zeros
        const uint4 zero = make_uint4(0u, 0u, 0u, 0u);
        for (int i = p.first + tid; i < p.last; i += kTokThreads) stream_store(out + (size_t)i * 16, zero);
        if (single >= 0) store_elem<DT>(out_row, single, 0.0f);
        return;
    }
    const uint32_t single_bits = single >= 0 ? load_raw<DT>(in_row, single) : 0u;
    const int yb = rec.y - p.head;
    float unused = 0.0f;  // (the sum for an entropy, which comes from the partials here)
    for (int i0 = p.first; i0 < p.last; i0 += kFewUnroll * kTokThreads) {
        uint4 v[kFewUnroll];
#pragma unroll
        for (int u = 0; u < kFewUnroll; ++u) {
            const int i = i0 + u * kTokThreads + tid;
            if (i < p.last) v[u] = row_load<ANY, false>(body + (size_t)i * 16);
        }
#pragma unroll
        for (int u = 0; u < kFewUnroll; ++u) {
            const int i = i0 + u * kTokThreads + tid;
            if (i < p.last) {
                float f[EPV];
                unpack<DT>(v[u], f);
                backward_vec<EPV, false>(f, -g, row_max, nls2, unused);
                stream_store(out + (size_t)i * 16, pack<DT>(f));
                // the chosen column gets +g from the thread that stored its vector (same thread, same address: program order)
                if (yb >= 0 && yb / EPV == i) store_elem<DT>(out, yb, -g * exp2_hw(fmaf(zy - row_max, kLog2e, nls2)) + g);
            }
        }
    }
    if (single >= 0) {
        float f[1] = {raw_to_float<DT>(single_bits)};
        backward_vec<1, false>(f, -g, row_max, nls2, unused);
        store_elem<DT>(out_row, single, single == rec.y ? f[0] + g : f[0]);
    }
}

// ---------------------------------------------------------------------------------------
// host side

constexpr int64_t kFewMaxRows = 256;  // (their partials fit the scratch area, and the last workgroup has a thread for each)
constexpr int64_t kFewPartBytes = 8192;

// Which batches come here, and parts per row: two workgroups per compute unit in all (four: 64 / 128 / 170 rows of bfloat16 x
// 151,936, the last two of which lie beyond the line, 24.2 / 30.0 / 31.3 us instead of 22.0 / 25.0 / 29.1), parts of at least 8 KiB,
// two at least.  A row of its own costs a
// compute unit the same however many other units are busy, while here all of them together read the batch twice and
// write it, so the line is one of bytes.  It lies where a batch of which every token counts is no slower (us, row kernel / here,
// every token / 9 in 16): bfloat16 64 x 151,936 (19 MB) 28.9 / 22.6, 29.3 / 22.0; 250 x 32,000 (16 MB) 25.2 / 21.0; 256 x 65,536
// (34 MB) 25.1 / 25.2; 150 x 151,936 (46 MB) 30.5 / 32.0; 170 (52 MB) 30.8 / 34.7, 32.6 / 29.1; 256 x 90,000 (46 MB) 27.6 / 31.7.
// Rows beyond the registers cost the one unit more: fp32 40 x 151,936 35.4 / 20.8, 64: 39.6 / 21.2, 100 (61 MB) 39.5 / 35.6,
// 110 (67 MB) 41.1 / 39.4.
int few_rows_parts(const LossArgs &a)
{
    const int64_t row_bytes = a.V * (a.dt == A3PO_F32 ? 4 : 2);
    const int64_t most_bytes = (row_bytes > (int64_t)kMaxVec * kRowThreads * 16 ? 64 : 32) << 20;
    // (the batch first: most calls need not ask for the device)
    if (a.T <= 0 || a.T > kFewMaxRows || row_bytes < 2 * kFewPartBytes || a.T * row_bytes > most_bytes) return 0;
    const GemmGrid chip = gemm_grid();
    const int64_t cus = (int64_t)chip.nxcd * chip.per_xcd;
    if (a.T > cus) return 0;
    int64_t parts = 2 * cus / a.T;
    if (parts > row_bytes / kFewPartBytes) parts = row_bytes / kFewPartBytes;
    return (int)(parts < 32 ? parts : 32);
}

template <typename DT, bool ENT, bool ANY>
static hipError_t launch_few_rows_t(const LossArgs &a, int parts, hipStream_t s)
{
    const unsigned grid = (unsigned)(a.T * parts + 1);
    hipLaunchKernelGGL((few_rows_partials_kernel<DT, ENT, ANY>), dim3(grid), dim3(kTokThreads), 0, s, a, parts);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((few_rows_gradient_kernel<DT, ENT, ANY>), dim3(grid), dim3(kTokThreads), 0, s, a, parts);
    return hipGetLastError();
}

template <typename DT>
static hipError_t launch_few_rows_dt(const LossArgs &a, int parts, hipStream_t s)
{
    // (whole vectors of the logits are aligned where every row's first line of the gradient begins a vector of them)
    const bool any = ((reinterpret_cast<uintptr_t>(a.z) ^ reinterpret_cast<uintptr_t>(a.dz)) & 15u) != 0;
    if (a.ent_out) return any ? launch_few_rows_t<DT, true, true>(a, parts, s) : launch_few_rows_t<DT, true, false>(a, parts, s);
    return any ? launch_few_rows_t<DT, false, true>(a, parts, s) : launch_few_rows_t<DT, false, false>(a, parts, s);
}

hipError_t launch_few_rows_loss(const LossArgs &a, int parts, hipStream_t s)
{
    if (a.T * parts > (int64_t)(kLossScratchBytes / sizeof(float4)) || a.T > kTokThreads) return hipErrorInvalidValue;
    return a.dt == A3PO_F32 ? launch_few_rows_dt<F32>(a, parts, s) : launch_few_rows_dt<Bf16>(a, parts, s);
}

}  // namespace a3po
