// Host-side launch interface between the C ABI (a3po_api.hip) and the kernel files.
#pragma once

#include <cmath>
#include <mutex>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "a3po.h"

namespace a3po {

struct TokenRecord;

struct LossArgs {
    const void *z;
    void *dz;
    int dt;  // a3po_dtype
    int64_t T, V, ld;
    const int32_t *chosen;
    const float *lb;
    const int32_t *versions;
    int32_t current_version;
    const float *adv;
    const uint8_t *mask;
    float clip_eps;
    float denom;
    float *logp_out;
    float *prox_out;  // nullable
    float *loss_out;
    a3po_stats *stats_out;  // nullable
    int prox_mode = 0;               // a3po_prox_mode
    const float *prox_in = nullptr;  // [T], A3PO_PROX_GIVEN only
    float *ent_out = nullptr;        // [T] policy entropy, nullable
    float *iw_out = nullptr;         // [T] importance weights, nullable
    uint8_t *clipped_out = nullptr;  // [T] clip decisions, nullable
    const float *denom_dev = nullptr;  // device [1], overrides denom when set
    int accumulate = 0;              // add to loss_out / stats_out instead of overwriting
    // workspace carve-up
    void *ws_header;
    TokenRecord *ws_records;  // [T], written by the prep kernel
    float *ws_obj;
    float *ws_iw;
    uint8_t *ws_flags;
    void *ws_scratch;               // kLossScratchBytes: per-workgroup partials of the prep and finish kernels
};

// Workspace of the loss path: header | TokenRecord[T] (16 bytes each) | obj[T] | iw[T] | flags[T] | scratch
struct LossWsLayout {
    size_t records, obj, iw, flags, scratch, total;
};

// The O(T) kernels before and after the row kernel run on up to kTokMaxBlocks workgroups of kTokBlockTokens tokens
// each (one workgroup for short batches); each leaves a partial of at most 64 bytes in the scratch area.
constexpr int kTokMaxBlocks = 256;
constexpr int kTokBlockTokens = 2048;
constexpr size_t kLossScratchBytes = (size_t)kTokMaxBlocks * 64;
inline LossWsLayout loss_ws_layout(int64_t T)
{
    auto up = [](size_t x) { return (x + 255) / 256 * 256; };
    const size_t t = (size_t)(T > 0 ? T : 0);
    LossWsLayout l;
    l.records = 256;
    l.obj = l.records + up(t * 16);
    l.iw = l.obj + up(t * sizeof(float));
    l.flags = l.iw + up(t * sizeof(float));
    l.scratch = l.flags + up(t);
    l.total = l.scratch + kLossScratchBytes;
    return l;
}

// points the workspace fields of `a` into a workspace laid out for T tokens
inline void carve_loss_ws(LossArgs &a, void *workspace, int64_t T)
{
    char *ws = static_cast<char *>(workspace);
    const LossWsLayout lay = loss_ws_layout(T);
    a.ws_header = ws;
    a.ws_records = reinterpret_cast<TokenRecord *>(ws + lay.records);
    a.ws_obj = reinterpret_cast<float *>(ws + lay.obj);
    a.ws_iw = reinterpret_cast<float *>(ws + lay.iw);
    a.ws_flags = reinterpret_cast<uint8_t *>(ws + lay.flags);
    a.ws_scratch = ws + lay.scratch;
}

hipError_t launch_loss_prep(const LossArgs &a, hipStream_t s);
hipError_t launch_loss_rows(const LossArgs &a, hipStream_t s);
// Parts that each row of a short batch is cut into for the kernels of a3po_few.hip (0: the batch takes the row kernel) ...
int few_rows_parts(const LossArgs &a);
// ... and the whole call (records, rows, loss and statistics) with that cut
hipError_t launch_few_rows_loss(const LossArgs &a, int parts, hipStream_t s);
hipError_t launch_loss_finish(const LossArgs &a, hipStream_t s);
hipError_t launch_count_tokens(const int32_t *chosen, const uint8_t *mask, int64_t T, int64_t V, float *denom_out,
                               int64_t *count_out, hipStream_t s);
// Workgroups of the histogram kernel.  Each adds its occupied slots to the one result when it is done, one atomic at a
// time and all workgroups in turn (some 12 ns each), so their number is bounded by what that costs against the values
// they count: one value per thread up to 192 workgroups, from some 280,000 values on 0.36 sqrt(T) of them.  64 bins,
// 192 / 512 / 1,024 / 2,048 workgroups: 131,072 values 10.8 / 14.4 / 14.4 / - us, 1,000,000: 20.0 / 18.9 / 27.8 / 48.2
// (360: 18.1), 4,000,000: 59 / 35 / 36 / 54 (768: 34), 16,000,000: 271 / 114 / 78 / 78, 64,000,000: 1,263 / 493 / 271 / 180.
constexpr int kHistThreads = 256;
inline int64_t histogram_blocks(int64_t T)
{
    const int64_t want = (T + kHistThreads - 1) / kHistThreads, root = (int64_t)(0.36 * std::sqrt((double)T));
    const int64_t most = root > 192 ? root : 192;
    return want < most ? want : most;
}
hipError_t launch_histogram(const float *values, const uint8_t *select, int64_t T, const float *edges, int nbins,
                            bool accumulate, int64_t *counts, hipStream_t s);

hipError_t launch_token_logprobs(const void *z, int dt, int64_t T, int64_t V, int64_t ld, const int32_t *chosen,
                                 float *logp, float *lse, void *chosen_logit, float *ent, hipStream_t s);
hipError_t launch_proximal_interp(const float *lb, const float *lt, const int32_t *versions, int32_t current_version,
                                  int64_t T, float *lp, float *alpha, hipStream_t s);
hipError_t launch_grpo_advantages(const float *rewards, int64_t S, int32_t G, float eps_adv, const int32_t *seq_id,
                                  int64_t T, float *adv, hipStream_t s);

// records (nullable): rows whose record says "not counted" are skipped (partials) / get zeros (combine)
hipError_t launch_shard_partials(const void *z, int dt, int64_t T, int64_t Vs, int64_t ld, const int32_t *chosen,
                                 int64_t v0, a3po_shard_partial *out, const TokenRecord *records, hipStream_t s);
hipError_t launch_shard_combine(const a3po_shard_partial *parts, int32_t P, int64_t T, const int32_t *chosen, int64_t V,
                                float *logp, float *lse, float *ent, const TokenRecord *records, hipStream_t s);
// the loss rows in three streaming passes (partials, merge, gradient bursts) for rows that do not fit on chip
// The row kernel and the gradient bursts hand out work through a 32-bit counter: item index = grid size + number
// of claims so far, and every workgroup makes one claim past the end.  Item counts above this bound are refused
// by the entry points (rows for the register-resident kernel, bursts for the streaming one).
constexpr int64_t kQueueMaxItems = ((int64_t)1 << 32) - ((int64_t)1 << 16);
int64_t shard_bwd_queue_items(int dt, int64_t T, int64_t Vs);  // bursts launch_shard_bwd_rows would queue (0: no queue)
// a.V is the shard width here; a.ws_records must come from a prep launch made with the full vocabulary size
hipError_t launch_shard_bwd_rows(const LossArgs &a, int64_t v0, const float *logp_theta, const float *lse, hipStream_t s);

// ---- bfloat16 contraction on the matrix cores (a3po_gemm.hip): C[m, n] = sum_k A(m, k) B(n, k) ---------------
// The products that exist, each with the layouts of its operands (see GemmArgs) and its epilogue:
enum GemmProduct {
    kGemmLse = 0,        // A rows, B rows: running (max, sum) per column n over the rows m -> partial; C untouched
    kGemmLseStore = 1,   // the same, and C^T (float) = the product
    kGemmSplitRows = 2,    // A panels, B slow rows: C (bfloat16) = the product; few tiles: the contraction is cut into
                           // slices (see gemm_slices)
    kGemmSplitPanels = 3,  // the same with B panels
    kGemmPanelsBf16 = 4,   // A panels, B panels: C^T (bfloat16) = the product
    kGemmPanelsF32 = 5     // the same in float, or += when accumulate is set
};

// An extent that is only known on the device when the launch is queued (the number of tokens that enter the loss):
// extent = clamp(*n - offset, 0, cap), or the host's value when n is null.
struct DynCount {
    const int64_t *n = nullptr;
    int64_t offset = 0, cap = 0;
};
__host__ __device__ inline int64_t dyn_extent(const DynCount &d, int64_t host_value)
{
    if (!d.n) return host_value;
    const int64_t v = *d.n - d.offset;
    return v < 0 ? 0 : (v > d.cap ? d.cap : v);
}

enum GemmDynDim { kDynNone = 0, kDynM = 1, kDynN = 2, kDynK = 3 };

// (see gemm_shape)
struct GemmShape {
    int mtiles, ntiles, ncol, ml, groups, rounds;
};

// (see gemm_cut)
struct GemmCut {
    GemmShape part[2];
    int tiles0;           // column tiles of part 0
    int64_t pairs0, pairs;
};

// Operand layouts (bfloat16, 16-byte aligned base, ld in elements):
//   rows         [M, K] row-major, row stride ld: the contracted index is the fast one
//   panels       panel layout (panel_offset) of [M, K]; ld = K extent of the buffer, rows padded to a multiple of 256
//   slow rows    [K, M] row-major, row stride ld (M a multiple of 64): the contracted index is the slow one
// Contracted positions beyond those that exist must hold zeros in a panel operand; beyond the last row of a slow-rows
// operand its last row is read again.
struct GemmArgs {
    const uint16_t *A;
    int64_t lda;
    const uint16_t *B;
    int64_t ldb;
    int64_t M, N, K;    // K a multiple of 64 (the others than kGemmLse*: of 128)
    int64_t k_rows;     // kGemmSplitRows: rows that B has
    void *C;            // row stride ldc elements; C^T: element (m, n) at C[n * ldc + m], M a multiple of the
    int64_t ldc;        // elements in 16 bytes
    float2 *partial;    // kGemmLse*: [slots][N] (max, sum) per column (see GemmShape), merged by the caller; room for
    int64_t room;       // this many entries, at least gemm_partial_entries(N)
    float *split;       // kGemmSplit*: room for split_max slices of M x N floats (overwritten)
    int split_max;
    int accumulate;     // kGemmPanelsF32
    int dyn_dim;        // GemmDynDim: which of M, N, K is replaced by dyn_extent(dyn, .) on the device (K: rounded up
    DynCount dyn;       // to 128; the host's M, N, K are then upper bounds).  A zero extent makes the launch a no-op.
    int nxcd, per_xcd;  // filled in by the launcher from the device: the persistent grid (nxcd x per_xcd workgroups)
    GemmCut cut;        // filled in by the launcher: kGemmLse* whose extents the host knows
};

// How the workgroups of an XCD (per_xcd of them) share the tile grid: a block of ml rows x ncol columns of tiles, whose
// operand tiles they share through that XCD's L2; the tile grid is cut into `groups` column groups of ncol tiles and
// `rounds` of ml tile rows.  Four columns where there are enough of them (8 x 4 tiles on 32 compute units); up to three,
// or five, six or nine, go as blocks of one to three columns, whose rows take the workgroups that this frees, and rows that
// would leave XCDs without a block are cut into more rounds, whose columns then take them (groups of different widths:
// gemm_cut).  More blocks than XCDs for that would be a second round for some of them: 16 x 12 tiles as 9
// blocks of 6 x 5 took two rounds for the one of 6 blocks of 8 x 4 (3,000 tokens x 4,096 x 4,000: 160 us, now 110).  A
// launch with the log-sum-exp epilogue leaves one partial per column in each of nxcd * ml slots (slot = xcd * ml + row of
// the block) that had a tile of that column.
// (A fixed 8 x 4 block left three workgroups in four idle for a single column of tiles: log-probs of 200 tokens x
// 4,096 x 151,936 925 us so, 333 us with blocks of 32 x 1; weight gradient with 6 tile rows 500 against 424 us.)
constexpr int kGemmTile = 256;  // tile edge, both sides
constexpr int kGemmColTiles = 4;
__host__ __device__ inline GemmShape gemm_shape(int64_t M, int64_t N, int nxcd, int per_xcd)
{
    GemmShape s;
    s.mtiles = (int)((M + kGemmTile - 1) / kGemmTile);
    s.ntiles = (int)((N + kGemmTile - 1) / kGemmTile);
    s.groups = (s.ntiles + kGemmColTiles - 1) / kGemmColTiles;
    s.ncol = (s.ntiles + s.groups - 1) / s.groups;
    s.ml = per_xcd / s.ncol > 0 ? per_xcd / s.ncol : 1;
    s.rounds = (s.mtiles + s.ml - 1) / s.ml;
    if (nxcd / s.groups > s.rounds) s.rounds = nxcd / s.groups;  // fewer blocks than XCDs: as many as do not exceed them
    s.ml = (s.mtiles + s.rounds - 1) / s.rounds;
    s.rounds = (s.mtiles + s.ml - 1) / s.ml;
    s.ncol = per_xcd / s.ml < s.ntiles ? per_xcd / s.ml : s.ntiles;
    s.groups = (s.ntiles + s.ncol - 1) / s.ncol;
    return s;
}

// Cut of a tile grid for the products whose columns are tokens (kGemmLse*): up to two runs of column groups of different
// widths, each with the blocks of rows that its width leaves room for; pairs are counted through both.  The columns are dealt
// to as many groups of four as they need, or to one group less of four and five, as evenly as they go, and the cut with the
// fewest tiles for the busiest workgroup is taken (the plain shape among them, which wins ties).  5 / 7 / 10 / 11 / 13 / 17
// columns of 594 tile rows then take 13 / 17 / 25 / 27 / 32 / 41 rounds of tiles for the 15 / 19 / 29 / 29 / 38 / 47 of equal
// groups.  A cut whose partials do not fit the `room` entries there are is left out.
// Log-probs of 1,100 / 1,700 / 2,400 / 3,200 / 4,200 tokens x 1,536 x 151,936 552 / 730 / 1,121 / 1,422 / 1,876 us with equal
// groups, 502 / 700 / 1,011 / 1,280 / 1,634 so.
__host__ __device__ inline int64_t gemm_cut_entries(const GemmCut &c, int64_t N, int nxcd)
{
    const int64_t n0 = (int64_t)c.tiles0 * kGemmTile < N ? (int64_t)c.tiles0 * kGemmTile : N;
    return (int64_t)nxcd * (c.part[0].ml * n0 + c.part[1].ml * (N - n0));
}
__host__ __device__ inline GemmCut gemm_plain_cut(const GemmShape &s)
{
    GemmCut c;
    c.part[0] = c.part[1] = s;
    c.part[1].ntiles = c.part[1].ml = 0;  // (empty)
    c.tiles0 = s.ntiles;
    c.pairs0 = c.pairs = (int64_t)s.groups * s.rounds;
    return c;
}
__host__ __device__ inline GemmCut gemm_cut(int64_t M, int64_t N, int nxcd, int per_xcd, int64_t room)
{
    GemmCut best = gemm_plain_cut(gemm_shape(M, N, nxcd, per_xcd));
    const int nt = best.part[0].ntiles, mt = best.part[0].mtiles;
    const int up = (nt + 3) / 4;
    for (int g = up; nt > 4 && per_xcd >= 8 && best.pairs > nxcd && g >= 1 && g >= up - 1; --g) {
        const int w = nt / g, more = nt % g;  // `more` groups of w + 1 columns, the others of w
        if (w + (more > 0) > 5) continue;
        GemmCut c;
        for (int i = 0; i < 2; ++i) {
            GemmShape &p = c.part[i];
            p.mtiles = mt;
            p.ncol = w + 1 - i;
            p.groups = i ? g - more : more;
            p.ntiles = p.groups * p.ncol;
            p.rounds = (mt + per_xcd / p.ncol - 1) / (per_xcd / p.ncol);
            p.ml = (mt + p.rounds - 1) / p.rounds;
        }
        c.tiles0 = c.part[0].ntiles;
        c.pairs0 = (int64_t)c.part[0].groups * c.part[0].rounds;
        c.pairs = c.pairs0 + (int64_t)c.part[1].groups * c.part[1].rounds;
        if ((c.pairs + nxcd - 1) / nxcd < (best.pairs + nxcd - 1) / nxcd && gemm_cut_entries(c, N, nxcd) <= room) best = c;
    }
    return best;
}

// Slices of a kGemmSplit* launch.  A product with fewer tiles than compute units (or a last round of tiles that fills
// few of them) leaves the chip idle for its whole contracted length, so the contraction is cut into slices that are
// work items of their own; their fp32 results are added in a fixed order by a second kernel.  The number of slices is
// the one with the least predicted time among those that fill one to four rounds of the grid, in units of 0.1 us:
// 3.2 us per 128 contracted elements and round, 4 us of epilogue per round, and 0.13 us of memory traffic per slice of
// a tile (256 KiB written and read back at 4 TB/s).  (560 x 1,536 over 151,936: 18 tiles, 2.4 ms in one piece, 0.30 +
// 0.014 ms as 14 slices; 512 tiles, two full rounds, stay whole: a second slice would only add its traffic.)
__host__ __device__ inline int gemm_slices(int64_t tiles, int64_t quads, int workgroups, int split_max)
{
    if (tiles > 2 * workgroups) return 1;  // (two slices would need more than four rounds)
    const int t = (int)tiles, q = (int)quads;
    auto cost = [&](int n) {
        const int rounds = (t * n + workgroups - 1) / workgroups;
        return rounds * ((q + n - 1) / n * 32 + 40) + (n > 1 ? n * t * 13 / 10 : 0);
    };
    int best = 1, least = cost(1);
    for (int k = 1; k <= 4; ++k) {
        int n = k * workgroups / t;
        n = n < split_max ? n : split_max;
        n = n < q ? n : q;
        const int c = n > 1 ? cost(n) : least;
        if (c < least) {
            least = c;
            best = n;
        }
    }
    return best;
}

// Panel layout of a bfloat16 operand of the contraction kernel: the matrix is cut into blocks of 256 rows x 32
// contracted elements - what one stage of the kernel consumes -, each stored as 256 rows x 64 bytes = 16 KiB
// contiguous; blocks of one 256-row band follow each other along K.  A direct load of the kernel (16 rows x 64
// bytes) is then 1 KiB of contiguous memory, eight whole 128-byte lines, instead of 16 half lines a row apart, and
// no power-of-two row stride maps a stage onto a few memory channels.  Element offset of (row, k), kext = K extent:
__host__ __device__ inline int64_t panel_offset(int64_t row, int64_t k, int64_t kext)
{
    return ((row >> 8) * (kext >> 5) + (k >> 5)) * 8192 + (row & 255) * 32 + (k & 31);
}
inline size_t panel_elements(int64_t rows, int64_t kext) { return (size_t)((rows + 255) / 256 * 256) * (size_t)kext; }

// Raises a kernel's dynamic-LDS limit once per device (the attribute belongs to the device's copy of the kernel),
// race-free: the first call on a device sets it under the lock, later calls only look at the flag.  One state
// object per kernel variant.
struct LdsLimitState {
    std::mutex lock;
    bool done[64] = {};
};
inline hipError_t ensure_lds_limit(const void *kernel, int bytes, LdsLimitState &st)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> guard(st.lock);
    if (!st.done[dev]) {
        e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (e != hipSuccess) return e;
        st.done[dev] = true;
    }
    return hipSuccess;
}

struct GemmGrid {
    int nxcd, per_xcd;
};
constexpr int kGemmMaxBlocks = 256;
GemmGrid gemm_grid();
// (max, sum) partials of up to N columns: nxcd * ml slots of N entries, at most 256 / ncol slots, and plain blocks
// (gemm_shape) of fewer than four columns exist only up to 256 (one), 512 (two) and 2,304 columns (three: 3, 5, 6 or 9
// tiles).  Cuts of two widths (gemm_cut) have groups of three columns, of 80 slots each, at 7, 10 and 11 tiles as well (4 + 3,
// 4 + 3 + 3, 4 + 4 + 3 of many rows), which this size happens to have room for; 3 + 2 at 5 tiles and 4 + 3 + 3 + 3 at 13 it has
// not, and gemm_cut, which checks each against the room there is (gemm_cut_entries), takes 5 and 5 + 4 + 4.
inline size_t gemm_partial_entries(int64_t N)
{
    auto upto = [&](int64_t slots, int64_t most) { return (size_t)(slots * (N < most ? N : most)); };
    size_t e = upto(kGemmMaxBlocks / 4, N);
    for (size_t o : {upto(kGemmMaxBlocks, 256), upto(kGemmMaxBlocks / 2, 512), upto(kGemmMaxBlocks / 3, 2304)}) e = o > e ? o : e;
    return e;
}
hipError_t launch_gemm(const GemmArgs &args, int product, hipStream_t s);

// Tiles of the few-token kernel: nfull whole tiles of kFewRows vocabulary entries, one for each compute unit and round, then
// those of the last round, each of last_blocks row blocks of 16: as many as an even share of them needs, or 16 (whole tiles
// again, on fewer units) where that is more than `most`.
constexpr int kFewWaves = 8;
constexpr int kFewRows = 32 * kFewWaves;
struct FewTiles {
    int nfull, ntiles, last_blocks, slots;
};
inline FewTiles few_tiles(int64_t V, int64_t cus, int most = 2 * kFewWaves)
{
    const int64_t blocks = (V + 15) / 16, rounds = (blocks - 1) / (2 * kFewWaves * cus), left = blocks - rounds * 2 * kFewWaves * cus;
    FewTiles f;
    f.last_blocks = (int)((left + cus - 1) / cus);
    if (f.last_blocks > most) f.last_blocks = 2 * kFewWaves;
    f.nfull = (int)(rounds * cus);
    f.ntiles = f.nfull + (int)((left + f.last_blocks - 1) / f.last_blocks);
    f.slots = (int)(f.ntiles < cus ? f.ntiles : cus);
    return f;
}
// Up to this many tokens the last round is always spread; beyond, where the products bind, only if no wavefront needs a second
// row block: with nine to fifteen blocks a tile every unit multiplies whole tiles' worth, and reads all the hidden rows, for part
// of one.  Whole tiles / spread, us: 200 tokens x 4,096 x 73,628 (2 blocks) 210 / 186, 98,204 (8) 224 / 207, 102,300 (9) 229 / 237,
// 118,684 (13) 244 / 249, 126,876 (15) 252 / 256; 200 x 768 x 110,492 (11) 54.7 / 57.1; 256 x 2,048 x 53,000 (13, no round before) 57.5 /
// 60.3; 160 x 4,096 x 102,300 (9) 205 / 200, 118,684 218 / 215, 160 x 1,024 x 118,684 56.5 / 57.2.
constexpr int kFewSpreadTokens = 192;
inline FewTiles few_tiles_of(int64_t T, int64_t V, int64_t cus)
{
    return few_tiles(V, cus, T <= kFewSpreadTokens ? 2 * kFewWaves : kFewWaves);
}

size_t lmhead_workspace_bytes(int64_t T);
hipError_t launch_fused_lmhead_logprob(const void *hidden, const void *weight, int64_t T, int64_t H, int64_t V,
                                       const int32_t *chosen, float *logp, float *lse, void *workspace, hipStream_t s);

// merges the (max, sum) partials of a token, adds the chosen logit (a dot product) and writes lse and log pi
// (room: as given to the contraction; T is an upper bound when `count` names a device-side token count; slots > 0: that many
// partials per token, all of them written, instead of those of a contraction)
hipError_t launch_lmhead_lse_finish(const void *hidden, const void *weight, int64_t T, int64_t H, int64_t V,
                                    const int32_t *chosen, const float2 *partial, float *logp,
                                    float *lse, hipStream_t s, int64_t room, DynCount count = DynCount(), int slots = 0);

size_t lmhead_bwd_workspace_bytes(int64_t T, int64_t V, int64_t H);

}  // namespace a3po
