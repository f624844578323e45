// Per-token work of a call (O(T)) that its kernels share: packing the records, the header, the loss and its statistics.
#pragma once

#include "a3po_common.h"
#include "a3po_launch.h"

namespace a3po {

constexpr int kTokThreads = 1024;
constexpr int kTokWaves = kTokThreads / kWave;

// Counts of a range of tokens: those that enter the loss (mask != 0 and a valid chosen id), and those with
// mask != 0 and an id outside [0, V).
struct PrepPartial {
    long long cnt, bad;
};

// Packs the inputs of tokens [t_begin, t_end) into one 16-byte record each for the row kernel (y = -1 when the
// token does not enter the loss) and counts them; the totals of the workgroup are returned to thread 0.
__device__ __forceinline__ PrepPartial pack_records(const int32_t *chosen, const uint8_t *mask, const float *lb,
                                                    const int32_t *versions, const float *adv, const float *prox_in,
                                                    int64_t t_begin, int64_t t_end, int64_t V, TokenRecord *records)
{
    __shared__ long long s_cnt[kTokWaves], s_bad[kTokWaves];
    long long cnt = 0, bad = 0;
    for (int64_t t = t_begin + threadIdx.x; t < t_end; t += kTokThreads) {
        const bool m = mask[t] != 0;
        const int32_t y = chosen[t];
        const bool ok = y >= 0 && (int64_t)y < V;
        cnt += (m && ok) ? 1 : 0;
        bad += (m && !ok) ? 1 : 0;
        TokenRecord r;
        r.y = (m && ok) ? y : -1;
        // a given proximal log-prob rides in the version slot; the coupled objective needs neither
        r.ver = prox_in ? __float_as_int(prox_in[t]) : (versions ? versions[t] : 0);
        r.lb = lb[t];
        r.A = adv[t];
        records[t] = r;
    }
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        cnt += __shfl_xor(cnt, off, kWave);
        bad += __shfl_xor(bad, off, kWave);
    }
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    if (lane == 0) {
        s_cnt[wave] = cnt;
        s_bad[wave] = bad;
    }
    __syncthreads();
    PrepPartial p = {0, 0};
    if (threadIdx.x == 0) {
        for (int w = 0; w < kTokWaves; ++w) {
            p.cnt += s_cnt[w];
            p.bad += s_bad[w];
        }
    }
    return p;
}

// Header of a call: 1/N with N the number of counted tokens, or the caller's denominator when it is positive;
// the counts for the statistics; the row kernel's work queue starts empty.
__device__ __forceinline__ void write_header(PrepPartial total, float denom, WsHeader *hdr)
{
    const float n = denom > 0.0f ? denom : (float)total.cnt;
    hdr->inv_n = n > 0.0f ? 1.0f / n : 0.0f;
    hdr->n_as_float = n;
    hdr->n_counted = total.cnt;
    hdr->n_bad = total.bad;
    *row_queue_of(hdr) = 0u;
}

// Totals of the finish pass over a range of tokens.
struct FinishTotals {
    double sum, esum;     // sum of obj and of the entropies over counted tokens
    long long clip, neg;  // clipped tokens, tokens with negative staleness
    float lo, hi;         // extrema of the importance weight
};

static_assert(sizeof(FinishTotals) <= 64 && sizeof(PrepPartial) <= 64, "a partial is at most 64 bytes of the scratch area");

// Totals of the workgroup's threads, in thread 0 (a fixed tree: repeated runs agree bit for bit).
// (The last sum goes four wavefronts at a time: all sixteen at once are 160 registers, which few_rows_gradient_kernel, of whose
// workgroups only one gets here, had to make room for: 127 or 128 registers and, with the entropy, 24 spilled; now 44 to 52.
// That kernel, with the entropy: 64 rows of bfloat16 x 151,936 9.6 -> 8.6 us, 256 x 32,000 8.9 -> 7.0, 100 of fp32 x 151,936
// 14.7 and 14.8.)
__device__ __forceinline__ FinishTotals block_totals(FinishTotals t)
{
    __shared__ FinishTotals s_tot[kTokWaves];
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        t.sum += __shfl_xor(t.sum, off, kWave);
        t.esum += __shfl_xor(t.esum, off, kWave);
        t.clip += __shfl_xor(t.clip, off, kWave);
        t.neg += __shfl_xor(t.neg, off, kWave);
        t.lo = fminf(t.lo, __shfl_xor(t.lo, off, kWave));
        t.hi = fmaxf(t.hi, __shfl_xor(t.hi, off, kWave));
    }
    if ((threadIdx.x & (kWave - 1)) == 0) s_tot[threadIdx.x / kWave] = t;
    __syncthreads();
    FinishTotals tot = {0.0, 0.0, 0, 0, INFINITY, -INFINITY};
    if (threadIdx.x == 0) {
#pragma unroll 4
        for (int w = 0; w < kTokWaves; ++w) {
            tot.sum += s_tot[w].sum;
            tot.esum += s_tot[w].esum;
            tot.clip += s_tot[w].clip;
            tot.neg += s_tot[w].neg;
            tot.lo = fminf(tot.lo, s_tot[w].lo);
            tot.hi = fmaxf(tot.hi, s_tot[w].hi);
        }
    }
    return tot;
}

// loss_out / stats_out from the totals of the whole call (overwritten, or merged into what earlier micro-batches of
// the same update left there)
__device__ __forceinline__ void write_loss_and_stats(const FinishTotals &tot, bool have_entropy, const WsHeader *hdr,
                                                     float *loss_out, a3po_stats *stats, int accumulate)
{
    const float share = (float)(-(tot.sum * (double)hdr->inv_n));
    *loss_out = accumulate ? *loss_out + share : share;
    if (!stats) return;
    a3po_stats o;
    o.n_tokens = hdr->n_counted;
    o.n_clipped = tot.clip;
    o.n_bad_index = hdr->n_bad;
    o.n_negative_staleness = tot.neg;
    o.iw_min = tot.lo;
    o.iw_max = tot.hi;
    o.entropy_mean = (have_entropy && hdr->n_counted > 0) ? (float)(tot.esum / (double)hdr->n_counted) : 0.0f;
    o.reserved = 0.0f;
    if (accumulate) {
        const a3po_stats p = *stats;
        const long long n = p.n_tokens + o.n_tokens;
        o.entropy_mean = (have_entropy && n > 0)
                             ? (float)(((double)p.entropy_mean * (double)p.n_tokens + tot.esum) / (double)n)
                             : 0.0f;
        o.n_tokens = n;
        o.n_clipped += p.n_clipped;
        o.n_bad_index += p.n_bad_index;
        o.n_negative_staleness += p.n_negative_staleness;
        o.iw_min = fminf(o.iw_min, p.iw_min);
        o.iw_max = fmaxf(o.iw_max, p.iw_max);
    }
    *stats = o;
}

}  // namespace a3po
