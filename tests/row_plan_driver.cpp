// How loss rows are dispatched (plan_rows), walked on the host over every row length up to beyond the registers:
//  - a kernel instance exists for the plan;
//  - all but its last sweep are full in every row, and what its sweeps do not hold fits the tail of single elements;
//  - rows of whole lines take as many threads as they were measured to be fastest with.
#include <cstdio>
#include <cstdlib>

#include "a3po_row_plan.h"

using namespace a3po;

static bool exists(int threads, int sweeps, bool ent)
{
#define A3PO_HAS(NT, N, PLAIN, WITH_ENT) \
    if (threads == NT && sweeps == N) return ent ? WITH_ENT : PLAIN;
    A3PO_ROW_INSTANCES(A3PO_HAS)
#undef A3PO_HAS
    return false;
}

template <typename DT>
static void walk(bool ent, bool edge, int64_t T)
{
    constexpr int64_t EPV = DT::kPerVec, E = DT::kBytes;
    float dummy;
    for (int64_t V = 1; V <= 190000; ++V) {
        LossArgs a = {};
        a.z = reinterpret_cast<const void *>((uintptr_t)(4096 + (edge ? E : 0)));
        a.dz = reinterpret_cast<void *>((uintptr_t)(8192 + (edge ? E : 0)));
        a.V = V;
        a.ld = (V * E + 127) / 128 * 128 / E;
        a.T = T;
        a.ent_out = ent ? &dummy : nullptr;
        const RowPlan p = plan_rows<DT>(a, 256);
        auto fail = [&](const char *what) {
            std::printf("%s: V %lld, %d bytes, entropy %d, edge %d: %d threads, %d sweeps\n", what, (long long)V,
                        DT::kBytes, ent, edge, p.threads, p.sweeps);
            std::exit(1);
        };
        if (p.edge != edge) fail("cut or not");
        if (p.kind == RowPlan::kLong) {
            if (V <= kMaxVec * 1024 * EPV) fail("a row that fits the registers taken as a long one");
            continue;
        }
        if (p.kind != RowPlan::kRegisters || !exists(p.threads, p.sweeps, ent)) fail("no such kernel");
        const int64_t full = (int64_t)(p.sweeps - 1) * p.threads, room = (int64_t)p.sweeps * p.threads;
        if (!edge) {
            const int64_t nvec = (V + EPV - 1) / EPV;
            if (!(full < nvec && nvec <= room)) fail("sweeps");
        }
        for (int64_t head = 0; edge && head < kLineBytes / E; ++head) {
            const int64_t h = head < V ? head : V, body = (V - h) / EPV, held = body < room ? body : room;
            if (held < full) fail("a sweep that is not full");
            if (V - h - held * EPV > p.threads - kEdgeTail0) fail("a tail that is too long");
        }
        const bool few = T <= (ent ? 512 : 768);
        const int64_t most = 1024 * (ent ? (few ? 104 : E == 4 ? 65 : 72) : (few ? 48 : E == 4 ? 40 : 42));
        if (!edge && p.threads != (V * E <= 16384 ? 256 : V * E <= most ? 512 : 1024)) fail("threads");
    }
}

// Forward-only rows, 256 compute units: counts between two and five rows per unit, rows a multiple of 256 KiB apart and
// short rows were measured slower with 512 threads (up to 1.16 and 1.6 times as long).
static void forward_rows()
{
    const struct {
        int64_t T, row, stride;
        bool ent;
        int want;
    } rows[] = {
        {1, 300 * 1024, 300 * 1024, false, 512},      {256, 16 * 1024, 16 * 1024, true, 512},
        {300, 297 * 1024, 297 * 1024, true, 512},     {400, 256 * 1024, 256 * 1024, false, 256},
        {513, 200 * 1024, 200 * 1024, false, 256},    {768, 600 * 1024, 600 * 1024, false, 256},
        {1280, 600 * 1024, 600 * 1024, false, 256},   {1536, 297 * 1024, 297 * 1024, true, 512},
        {1536, 64 * 1024, 64 * 1024, false, 256},     {2048, 297 * 1024, 297 * 1024, false, 256},
        {10240, 297 * 1024, 297 * 1024, false, 512},  {10240, 297 * 1024, 297 * 1024, true, 256},
        {10240, 256 * 1024, 256 * 1024, false, 256},  {10240, 32 * 1024, 32 * 1024, false, 256},
    };
    for (const auto &r : rows)
        if (logprob_row_threads(r.T, r.row, r.stride, r.ent, 256) != r.want) {
            std::printf("forward rows: %lld of %lld bytes, entropy %d\n", (long long)r.T, (long long)r.row, r.ent);
            std::exit(1);
        }
}

int main()
{
    forward_rows();
    for (bool ent : {false, true})
        for (bool edge : {false, true})
            for (int64_t T : {1, 512, 768, 769, 100000}) {
                walk<F32>(ent, edge, T);
                walk<Bf16>(ent, edge, T);
            }
    std::puts("ok");
}
