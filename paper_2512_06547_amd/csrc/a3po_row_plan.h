// Which kernel of a3po_rows.hip takes the rows of a loss call (host code only: no kernel here, so that the rule can be
// walked by a program of its own).
#pragma once

#include "a3po_common.h"
#include "a3po_launch.h"

namespace a3po {

constexpr int kRowThreads = 1024;
constexpr int kMaxVec = 20;        // 16-byte vectors per thread that the fused kernel can hold
constexpr int kLineBytes = 128;
constexpr int kEdgeTail0 = kWave;  // first thread of a cut row's tail (see EdgeSpan)

inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// How the rows of a call are handled.
struct RowPlan {
    enum Kind { kRegisters, kLong, kElements } kind;
    bool edge;   // cut rows at the lines of the gradient (see EdgeSpan)
    int threads, sweeps;  // kRegisters: template arguments NT and NSWEEP
};

// Rows whose bases are multiples of 16 bytes and whose stride is a multiple of 128 are taken whole; others are cut at
// the lines of the gradient.  (A stride of whole vectors could be taken whole too, but the cut makes every store cover
// whole lines: 8,192 rows of bfloat16 x 32,008 / 100,360 / 151,944 210 / 621 / 988 us whole, 199 / 564 / 875 us cut.)
//
// Threads per row.  Short rows need more of them in flight per compute unit than one or two workgroups of 1024: 256
// threads up to 16 KiB (8,192 rows of bfloat16 x 8,192: 119 us with 1024 threads, 67 so), then 512.  Where 512 ends depends
// on how many rows there are.  With no more than two (without the entropy three) per compute unit each is on its own, and
// 512 threads, of which a unit takes several at once, are faster at any length (250 / 400 / 512 rows of 41 to 104 KiB: 0.84 /
// 0.79 / 0.78 of the time with 1024; used up to 48 KiB, with the entropy 104).  With more of them the two cross, at
// different lengths for batches that all count, batches masked in runs (tails of sequences) and here and there; the line
// lies where none is more than 3 % slower (8,192 rows, time with 512 threads over that with 1024):
//                        all count / in runs / here and there
//   bfloat16             42 KiB 0.91 0.96 0.97    47 KiB  0.97 1.03 1.03
//   fp32                 40 KiB 0.99 0.96 0.93    44 KiB  1.04 1.00 1.01    47 KiB  1.04 1.05 1.04
//   bfloat16, entropy    72 KiB 0.83 0.96 1.03    80 KiB  0.87 1.00 1.06    98 KiB  0.93 1.04 1.09
//   fp32, entropy        65 KiB 0.90 0.98 1.03    72 KiB  0.94 1.02 1.07    98 KiB  1.05 1.07 1.11
// (with the entropy the temporaries do not fit beside a row in the 64 registers of two workgroups of 1024, which rows
// of up to four of their sweeps run as: those keep 512 threads).
//
// A row whose body needs more than kMaxVec sweeps goes through the long kernel, whose direct loads into LDS want
// 16-byte addresses: logits and gradient must then have the same alignment within 16 bytes.  What is left (a long row
// of which they do not) is taken element by element.
template <typename DT>
inline RowPlan plan_rows(const LossArgs &a, int cus)
{
    constexpr int64_t EPV = DT::kPerVec;
    const bool edge = !(aligned16(a.z) && aligned16(a.dz) && (a.ld * DT::kBytes) % kLineBytes == 0);
    const int64_t head_max = kLineBytes / DT::kBytes - 1;
    const int64_t least = (a.V > head_max ? a.V - head_max : 0) / EPV;  // body vectors of the row with the fewest
    const int64_t nvec = (a.V + EPV - 1) / EPV;
    auto sweeps = [&](int64_t nt) { return edge ? least / nt + 1 : (nvec + nt - 1) / nt; };
    if (sweeps(256) <= 4) return {RowPlan::kRegisters, edge, 256, (int)sweeps(256)};
    constexpr bool kF32 = DT::kBytes == 4;
    const bool few = a.T <= (a.ent_out ? 2 : 3) * (int64_t)cus;
    const int64_t most = 1024 * (a.ent_out ? (few ? 104 : kF32 ? 65 : 72) : (few ? 48 : kF32 ? 40 : 42));
    if (a.V * DT::kBytes <= most || (a.ent_out && sweeps(kRowThreads) <= 4))
        return {RowPlan::kRegisters, edge, 512, (int)sweeps(512)};
    if (sweeps(kRowThreads) <= kMaxVec) return {RowPlan::kRegisters, edge, kRowThreads, (int)sweeps(kRowThreads)};
    const bool same = ((reinterpret_cast<uintptr_t>(a.z) ^ reinterpret_cast<uintptr_t>(a.dz)) & 15u) == 0;
    return {same ? RowPlan::kLong : RowPlan::kElements, edge, kRowThreads, 0};
}

// the instances that plan_rows can ask for: threads, sweeps, without / with the entropy
#define A3PO_ROW_INSTANCES(X) \
    X(256, 1, 1, 1) X(256, 2, 1, 1) X(256, 3, 1, 1) X(256, 4, 1, 1) \
    X(512, 3, 1, 1) X(512, 4, 1, 1) X(512, 5, 1, 1) X(512, 6, 1, 1) X(512, 7, 0, 1) X(512, 8, 0, 1) X(512, 9, 0, 1) \
    X(512, 10, 0, 1) X(512, 11, 0, 1) X(512, 12, 0, 1) X(512, 13, 0, 1) \
    X(1024, 3, 1, 0) X(1024, 4, 1, 0) X(1024, 5, 1, 1) X(1024, 6, 1, 1) X(1024, 7, 1, 1) X(1024, 8, 1, 1) \
    X(1024, 9, 1, 1) X(1024, 10, 1, 1) X(1024, 11, 1, 1) X(1024, 12, 1, 1) X(1024, 13, 1, 1) X(1024, 14, 1, 1) \
    X(1024, 15, 1, 1) X(1024, 16, 1, 1) X(1024, 17, 1, 1) X(1024, 18, 1, 1) X(1024, 19, 1, 1) X(1024, 20, 1, 1)

// Threads per row of the forward-only kernel, five wavefronts per SIMD either way.  512
//  - where a row has a compute unit to itself, since it is bound by what that can have in flight (64 / 256 rows of 151,936
//    bfloat16 17.5 / 20.8 us with 256 threads, 13.3 / 16.5 with 512), and up to two rows per compute unit (300 rows of 150 to
//    600 KiB 0.92 to 1.02 of the time);
//  - for many long rows without the entropy (10,240 rows of 151,936 bfloat16 484 -> 470 us; 3,000 rows of 125 to 600 KiB
//    0.95 to 1.02 of the time, 1,800 and 2,048 up to 1.04);
//  - for long rows of which six fall to a compute unit that holds five of 256 threads at a time (1,536 rows of 125 to 600
//    KiB 0.91 to 1.00 of the time).
// 256 for all others: 513 to 1,280 rows of 100 to 600 KiB take up to 1.16 times as long with 512, many short ones 1.6;
// rows a multiple of 256 KiB apart, which meet on the same memory channels, 1.02 to 1.09 in the last three of these cases.
inline int logprob_row_threads(int64_t T, int64_t row_bytes, int64_t stride_bytes, bool entropy, int64_t cus)
{
    if (T <= cus) return 512;
    const bool is_long = row_bytes >= 112 * 1024, two = T <= 2 * cus, six = is_long && T > 5 * cus && T <= 6 * cus;
    const bool many = is_long && !entropy && T >= 11 * cus;
    return (two || six || many) && stride_bytes % (256 * 1024) != 0 ? 512 : 256;
}

}  // namespace a3po
