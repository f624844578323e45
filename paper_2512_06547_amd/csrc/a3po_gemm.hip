// bfloat16 contraction on the matrix cores for the LM-head path:  C(m, n) = sum_k A(m, k) B(n, k), fp32 accumulation
// (v_mfma_f32_16x16x32_bf16).  The products that exist (GemmProduct) differ in the layouts of their operands and in
// what happens to each 256 x 256 tile as it leaves the accumulators:
//   kGemmLse        folded into a running (max, sum) per column n over the rows m (the online log-sum-exp of the
//                   vocabulary when A is the LM-head weight and B the hidden states); C is not written
//   kGemmLseStore   the same, and the tile is also stored as fp32 (the logits of a token chunk, kept for the
//                   backward pass)
//   kGemmSplit*     stored as bfloat16 (the gradient of the hidden states), or as fp32 slices to be added up
//   kGemmPanelsBf16 stored as bfloat16 (the weight gradient of a batch whose tokens fit one contraction)
//   kGemmPanelsF32  stored as fp32, or added to what C holds (the weight gradient, summed over groups of tokens)
//
// Tiling.  A workgroup of 512 threads (8 wavefronts, two per SIMD) computes a 256 x 256 tile, each wavefront a
// 128 x 64 part = 8 x 4 MFMA tiles of 16 x 16 = 128 accumulator registers.  Two wavefronts per SIMD: while one
// waits (for the stage barrier, for its fragments) the other keeps the matrix core busy, which one wavefront with
// 256 accumulators cannot; the 16 x 16 x 32 instruction also draws less power per flop than the 32 x 32 x 16 one,
// and at these sizes the chip is power-limited (the clock falls as the matrix cores get busier).  In the 16 x 16
// result layout a lane owns one column n and 4 rows m of each MFMA tile, so a reduction over m is mostly per
// lane.
//
// K is walked in stages of 32 (one MFMA deep) through a ring of LDS buffers that direct global -> LDS loads
// (global_load_lds_dwordx4: lane l of a wavefront lands at lds_base + 16 l; no staging registers, no LDS write
// instructions) fill a few stages ahead.  Operand layouts and their LDS images: see Operand below.
//
// Schedule of stage i (32 MFMAs per wavefront).  At the top a wavefront waits for its own loads of stage i+1 and
// its own fragment reads, and all wavefronts meet at one barrier: stage i+1 is now visible and the slot of stage i
// is free.  The 8 row fragments live in one set of registers: each is re-read for stage i+1 right after its last
// use in stage i; the 4 column fragments, which every MFMA group of the stage needs, alternate between two sets.
// The 4 direct loads of stage i + kDmaStages go into the freed slot, spread over the stage.  The ring runs through
// a workgroup's whole sequence of tiles without a break: the refills of a tile's last stages already bring the
// next tile's first stages, so a tile's epilogue overlaps with their arrival (what it keeps in LDS beside the ring is accessed
// through lds_put and lds_get, for which the compiler waits for no direct load).
//
// Tile order.  One persistent workgroup per compute unit; the workgroups of an XCD (dispatch order deals
// workgroups round-robin over the XCDs) form a block of ml x ncol tiles (8 x 4 in the usual case, GemmShape) that
// share ml tiles of A and ncol tiles of B through that XCD's L2.  The tile grid is cut into such blocks ("pairs" of a
// column group and a row round); pair p = group * rounds + round, counted on through the groups of both widths where there
// are two (GemmCut), and each XCD takes a contiguous range of pairs, i.e. it sweeps down the rows of one column group before
// it moves to the next.  With kGemmLse* a workgroup therefore keeps its running (max, sum) in registers over a whole sweep
// and writes one partial per column per sweep.
//
// Results.  The logits and the weight gradient are stored transposed (element (m, n) at C[n ldc + m]): a lane's four
// accumulator values of one MFMA tile are four consecutive m of one n, which a staging tile in LDS puts together to whole
// lines (store_tile_lines).
// One of M, N, K may be known only on the device (DynCount): the launch is sized for the host's upper bound and
// every workgroup reads the extent first; beyond it there is nothing to do and it returns.
#include "a3po_common.h"
#include "a3po_launch.h"
#include "a3po_direct.h"
#include <type_traits>

namespace a3po {

constexpr int kGemmThreads = 512;
constexpr int kGemmWaves = kGemmThreads / kWave;

constexpr int kDmaStages = 4;
constexpr int kDmaK = 32;                                  // K elements per stage
constexpr int kDmaRowBytes = kDmaK * 2;                    // 64
constexpr int kDmaOperandBytes = kGemmTile * kDmaRowBytes; // 16,384
constexpr int kDmaStageBytes = 2 * kDmaOperandBytes;       // 32,768
constexpr int kDmaRingBytes = kDmaStages * kDmaStageBytes; // 131,072 of the compute unit's 163,840
constexpr int kGemmRedBytes = 2 * kGemmTile * (int)sizeof(float2);  // column partials of the two row halves
// per-wavefront staging tile of the store epilogues: 16 rows x 32 columns of fp32, rows 36 floats apart
constexpr int kStageLd = 36;
constexpr int kStageBytes = 16 * kStageLd * (int)sizeof(float);  // 2,304
constexpr int kGemmLdsBytes = kDmaRingBytes + kGemmRedBytes + kGemmWaves * kStageBytes;  // 153,600 of 163,840

// Accumulator layout of a wavefront: acc[a][b][i] is row a 16 + 4 (lane >> 4) + i, column b 16 + (lane & 15) of its
// 128 x 64 part of the tile.

// Folds the 32 rows this lane holds of column block b (8 MFMA tiles x 4 values) into the lane's running
// (max, sum).  Row offsets >= mlim lie past the last row (only in the last, ragged tile); mlim is relative to the
// lane's first row.  The accumulators are only read.
template <bool RAGGED>
__device__ __forceinline__ void fold_column(const f32x4_t (&acc)[8][4], int b, int mlim, float &run_m, float &run_s)
{
    float mx = -INFINITY;
#pragma unroll
    for (int a = 0; a < 8; ++a) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float v = acc[a][b][i];
            if (RAGGED && a * 16 + i >= mlim) v = -INFINITY;
            mx = fmaxf(mx, v);
        }
    }
    const float m_new = fmaxf(run_m, mx);
    float s = run_s * exp2_hw((run_m - m_new) * kLog2e);
#pragma unroll
    for (int a = 0; a < 8; ++a) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float v = acc[a][b][i];
            if (RAGGED && a * 16 + i >= mlim) v = -INFINITY;
            s += exp2_hw((v - m_new) * kLog2e);
        }
    }
    run_m = m_new;
    run_s = s;
}

// Element-wise store of a wavefront's part of a tile that reaches past M or N (rows / columns beyond are skipped): one
// accumulator register covers 4 rows x 16 consecutive columns.
template <typename DT>
__device__ __forceinline__ void store_tile_edge(const f32x4_t (&acc)[8][4], void *C, int64_t ldc, int64_t m0, int64_t n0,
                                                int64_t M, int64_t N, int wm, int wn, int lane)
{
    const int col0 = wn * 64 + (lane & 15);
    const int row0 = wm * 128 + 4 * (lane >> 4);
    const int rows_left = (int)(M - m0 < kGemmTile ? M - m0 : kGemmTile);
    const int cols_left = (int)(N - n0 < kGemmTile ? N - n0 : kGemmTile);
#pragma unroll
    for (int a = 0; a < 8; ++a) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = row0 + a * 16 + i;
            if (row >= rows_left) continue;
#pragma unroll
            for (int b = 0; b < 4; ++b)
                if (col0 + b * 16 < cols_left) store_elem<DT>(C, (m0 + row) * ldc + n0 + col0 + b * 16, acc[a][b][i]);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Adds a tile to C^T (fp32; element (m, n) at C[n * ldc + m]) through the memory side's adders.  M is a multiple of 4.
__device__ __forceinline__ void add_tile_transposed(const f32x4_t (&acc)[8][4], float *C, int64_t ldc, int64_t m0, int64_t n0,
                                                    int64_t M, int64_t N, int wm, int wn, int lane)
{
    const int col0 = wn * 64 + (lane & 15);
    const int row0 = wm * 128 + 4 * (lane >> 4);
    const int rows_left = (int)(M - m0 < kGemmTile ? M - m0 : kGemmTile);
    const int cols_left = (int)(N - n0 < kGemmTile ? N - n0 : kGemmTile);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        if (col0 + b * 16 >= cols_left) continue;
        float *col = C + (n0 + col0 + b * 16) * ldc + m0 + row0;
#pragma unroll
        for (int a = 0; a < 8; ++a) {
            if (row0 + a * 16 >= rows_left) continue;
#pragma unroll
            for (int i = 0; i < 4; ++i) unsafeAtomicAdd(col + a * 16 + i, acc[a][b][i]);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Store of C^T in whole 128-byte lines: 16 columns x 32 rows (fp32; bfloat16: 64) at a time go through this wavefront's
// staging tile in LDS, into which a lane's four values of an MFMA tile, consecutive m of one column, go as one write, and
// leave as 8 columns x 128 bytes per store instruction.  (LDS instructions of one wavefront execute in order: no waits or
// barriers between its writes and its reads.)
// Straight from the registers a store instruction covers 16 columns x 64 (bfloat16: 32) bytes, and the memory takes such
// pieces of lines far more slowly than whole ones: the weight gradient of 53 / 654 / 2,557 tokens (1,536 x 151,936, whose
// 467 MB of stores bound it) 193 / 385 / 950 us so, 163 / 335 / 905 with pieces of 64 bytes, 140 / 335 / 890 with lines.
// Non-temporal: nothing in this call reads the weight gradient again, and what it would displace from the caches is the
// weight (119 us at 53 tokens, and the next projection 137 instead of 167; no gain from 654 tokens on); the logits (a few GB
// per chunk) do not fit any cache (projection with stores of 2,557 tokens x 896 x 50,264 / 1,536 x 151,936 375 / 1,605 us
// before, 340 / 1,540 with lines that are not, 310 / 1,500 so).
// EDGE: the tile reaches past M or N; M is a multiple of the elements in 16 bytes.
template <typename DT, bool EDGE>
__device__ __forceinline__ void store_tile_lines(const f32x4_t (&acc)[8][4], void *C, int64_t ldc, int64_t m0, int64_t n0,
                                                 int64_t M, int64_t N, int wm, int wn, int lane, char *stage)
{
    constexpr int kTiles = 8 / DT::kBytes;  // MFMA tiles along m that make up a line
    constexpr int kPitch = kStageLd * (int)sizeof(float);
    char *put = stage + (lane & 15) * kPitch + (lane >> 4) * 4 * DT::kBytes;  // column lane & 15, rows 4 (lane >> 4) ..
    const char *get = stage + (lane >> 3) * kPitch + (lane & 7) * 16;         // column lane >> 3 (+ 8), 16 bytes of its line
    const int col0 = wn * 64 + (lane >> 3), row0 = wm * 128 + (lane & 7) * DT::kPerVec;
    char *out = reinterpret_cast<char *>(C) + ((n0 + col0) * ldc + m0 + row0) * DT::kBytes;
    const int64_t eight = 8 * ldc * DT::kBytes;
    const int rows_left = (int)(M - m0 < kGemmTile ? M - m0 : kGemmTile);
    const int cols_left = (int)(N - n0 < kGemmTile ? N - n0 : kGemmTile);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
#pragma unroll
        for (int a = 0; a < 8; a += kTiles) {
#pragma unroll
            for (int u = 0; u < kTiles; ++u) {
                const f32x4_t v = acc[a + u][b];
                if constexpr (DT::kBytes == 4) lds_put(put + u * 64, v);
                else lds_put(put + u * 32, f32x2_t{__uint_as_float(pack_bf16x2(v[0], v[1])), __uint_as_float(pack_bf16x2(v[2], v[3]))});
            }
            asm volatile("" ::: "memory");
#pragma unroll
            for (int pass = 0; pass < 2; ++pass) {
                const f32x4_t v = lds_get<f32x4_t>(get + pass * 8 * kPitch);
                if (!EDGE || (col0 + 16 * b + 8 * pass < cols_left && row0 + 16 * a < rows_left))
                    __builtin_nontemporal_store(v, reinterpret_cast<f32x4_t *>(out + (2 * b + pass) * eight + a * 16 * DT::kBytes));
            }
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// Plain store of a tile that lies inside C, with 16-byte stores: 16 rows x 32 columns at a time go through a staging
// tile in LDS that belongs to this wavefront alone (LDS instructions of one wavefront execute in order, so no waits
// or barriers are needed between its writes and its reads) and leave as 8 rows x 128 bytes (fp32) or 8 rows x 64
// bytes (bfloat16) per store instruction.
template <typename DT>
__device__ __forceinline__ void store_tile_wide(const f32x4_t (&acc)[8][4], void *C, int64_t ldc, int64_t m0, int64_t n0,
                                                int wm, int wn, int lane, float *stage)
{
    const int wcol = lane & 15, wrow = 4 * (lane >> 4);  // where this lane's accumulator registers sit in a 16 x 16 tile
    const int rrow = lane >> 3, rcol = (lane & 7) * 4;   // what it reads back: 4 consecutive columns of row rrow + 8 pass
#pragma unroll
    for (int a = 0; a < 8; ++a) {
#pragma unroll
        for (int bp = 0; bp < 2; ++bp) {  // column blocks 2 bp, 2 bp + 1
#pragma unroll
            for (int bb = 0; bb < 2; ++bb)
#pragma unroll
                for (int i = 0; i < 4; ++i) stage[(wrow + i) * kStageLd + bb * 16 + wcol] = acc[a][2 * bp + bb][i];
            asm volatile("" ::: "memory");
            const int64_t at = (m0 + wm * 128 + a * 16 + rrow) * ldc + n0 + wn * 64 + bp * 32 + rcol;
#pragma unroll
            for (int pass = 0; pass < 2; ++pass) {
                const float4 v = lds_get<float4>(stage + (rrow + 8 * pass) * kStageLd + rcol);
                if constexpr (DT::kBytes == 2) {
                    *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(C) + at + (int64_t)pass * 8 * ldc) =
                        make_uint2(pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w));
                } else {
                    *reinterpret_cast<float4 *>(reinterpret_cast<float *>(C) + at + (int64_t)pass * 8 * ldc) = v;
                }
            }
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// ---- operands -----------------------------------------------------------------------------------------------
// One stage of an operand is 256 rows (m or n) x 32 contracted elements = 16 KiB of LDS, brought in by 16 direct loads
// of 1 KiB, two per wavefront (load j of wavefront w is number 8 j + w); a fragment is the 16 rows x 32 elements that
// one MFMA takes, lane l holding row l & 15 and elements 8 (l >> 4) .. + 7.
//
// Contracted index fast (kRows, kPanels): a load covers 16 rows x 64 bytes; LDS row r is 64 bytes, its four 16-byte
// pieces permuted by (r >> 2) & 3 on the global side of the load, and a fragment is one 16-byte read per lane (16
// consecutive rows, same logical piece: 16 distinct bank groups).
//
// Contracted index slow (kSlowRows): LDS holds the stage as it lies in memory, contracted elements as rows, and
// ds_read_b64_tr_b16 transposes on the way out: within a group of 16 lanes, lane i receives as value j the element i % 4
// of the 8 bytes addressed by lane i / 4 + 4 j.  With lane s of group q pointing at row 8 q + s / 4 (+ 4 for the second
// read), columns 4 (s % 4) .., two reads give each lane 8 contracted elements of column lane & 15.  A load covers 8 rows x
// 128 bytes (whole lines); LDS is 4 blocks of [32 rows][128 bytes], the four 32-byte granules of row r permuted by
// (r >> 1) & 3, so that the 4 rows x 32 bytes of a lane group fall into distinct banks.
enum OperandLayout { kRows, kPanels, kSlowRows };

typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) bf16x4_t *lds_tr_ptr_t;

// (the __restrict__ parameters put the read into an alias scope of its own once this is inlined: without one the
// compiler waits for every direct load in flight, vmcnt(0), before each transposing read; the stage's own wait and
// barrier are what orders the two)
__device__ __forceinline__ bf16x4_t tr_half(lds_tr_ptr_t __restrict__ p) { return __builtin_amdgcn_ds_read_tr16_b64_v4bf16(p); }
__device__ __forceinline__ bf16x8_t tr_read(char *lo, char *hi)
{
    const bf16x4_t a = tr_half((lds_tr_ptr_t)lo), b = tr_half((lds_tr_ptr_t)hi);
    return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}

template <int L>
struct Operand {
    static constexpr bool kSlow = L == kSlowRows;
    const char *base;    // of the operand
    int64_t ld;          // elements
    int64_t extent;      // rows of the result on this operand's side
    uint32_t k_last;     // kSlowRows: last row that exists
    int wave, lane;
    const char *tile;    // of the current tile
    uint32_t off[2];     // this lane's byte offsets of its two loads

    __device__ __forceinline__ void init(const uint16_t *p, int64_t ld_, int64_t extent_, int64_t k_rows, int wave_, int lane_)
    {
        base = reinterpret_cast<const char *>(p);
        ld = ld_;
        extent = extent_;
        k_last = (uint32_t)(k_rows - 1);
        wave = wave_;
        lane = lane_;
    }
    // rows or columns past the end of the operand are clamped (computed, never written); rows of panels exist (padding)
    __device__ __forceinline__ void set_tile(int t)
    {
        // (a 256-row band of panels is as long as 256 rows)
        tile = base + (int64_t)t * kGemmTile * 2 * (kSlow ? 1 : ld);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int i = 8 * j + wave;
            if constexpr (!kSlow) {
                const int r = i * 16 + (lane >> 2), last = (int)(extent - 1 - (int64_t)t * kGemmTile);
                const uint32_t piece = (uint32_t)((lane & 3) ^ ((lane >> 4) & 3)) * 16u;
                off[j] = L == kPanels ? (uint32_t)r * 64u + piece : (uint32_t)min(r, last) * ((uint32_t)ld * 2u) + piece;
                // (known to the compiler, a panel offset would be added to the tile's base once, in vector registers, and
                // every load would need a 64-bit vector addition instead of a scalar base and this offset)
                if constexpr (L == kPanels) asm volatile("" : "+v"(off[j]));
            } else {
                const int block = min((i >> 2) * 64, (int)(extent - 64 - (int64_t)t * kGemmTile));
                const uint32_t granule = (uint32_t)(((lane & 7) >> 1) ^ ((lane >> 4) & 3));  // row = 8 (i & 3) + (lane >> 3)
                off[j] = (uint32_t)block * 2u + granule * 32u + (uint32_t)(lane & 1) * 16u;
            }
        }
    }
    // load j of stage st into the operand's 16 KiB at dst: a base that is the same for the wavefront, a 32-bit lane offset
    __device__ __forceinline__ void refill(char *dst, int j, uint32_t st) const
    {
        const char *src;
        if constexpr (!kSlow) {
            src = tile + st * (L == kPanels ? 16384u : (uint32_t)kDmaRowBytes) + off[j];
        } else {
            const uint32_t row0 = min(st * (uint32_t)kDmaK, k_last), row = min(8u * (wave & 3) + (uint32_t)(lane >> 3), k_last - row0);
            src = tile + (uint64_t)row0 * ((uint32_t)ld * 2u) + (row * ((uint32_t)ld * 2u) + off[j]);
        }
        dma16(src, dst + (8 * j + wave) * 1024);
    }
    // this lane's part of a fragment's address, for the fragments of a wavefront whose part of the stage begins at 16-row
    // block t0 (a multiple of 4), and fragment t from there in the stage at p
    __device__ __forceinline__ uint32_t lane_base(int t0) const
    {
        if constexpr (!kSlow) return t0 * 1024u + (uint32_t)(lane & 15) * kDmaRowBytes + (uint32_t)(((lane >> 4) ^ ((lane >> 2) & 3)) * 16);
        const int row = 8 * (lane >> 4) + ((lane & 15) >> 2);
        return t0 * 1024u + row * 128u + (lane & 3) * 8u + ((lane >> 3) & 1) * 32u;
    }
    static __device__ __forceinline__ bf16x8_t fragment(char *p, uint32_t lane0, int t)
    {
        if constexpr (!kSlow) return *reinterpret_cast<const bf16x8_t *>(p + lane0 + t * 1024);
        // granule t & 3 of rows 8 q + s / 4 is stored at granule (t & 3) ^ (s >> 3), of the rows 4 further at
        // that ^ 2: lane0 holds the place of granule 0, and an odd granule lies 32 bytes up or down from the even one
        char *q = p + (t >> 2) * 4096 + ((t & 1) ? lane0 ^ 32u : lane0);
        return tr_read(q + (t & 2) * 32, q + ((t & 2) ^ 2) * 32 + 512);
    }
};

// a value that is the same for the wavefront, in scalar registers (64-bit divisions leave theirs in vector registers)
__device__ __forceinline__ int64_t uniform64(int64_t v)
{
    return (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) |
                     (uint32_t)__builtin_amdgcn_readfirstlane((int)v));
}

// QUAD: K is a multiple of kDmaStages stages.  Then every tile starts in ring slot 0, the K loop is unrolled by
// the ring depth (all LDS addresses are constants) and the refill cursor moves once per kDmaStages stages.
// Otherwise the loop is unrolled by two (the column fragments alternate; the number of stages is even) and slot
// and cursor are tracked per stage.
//
// kGemmSplit* (QUAD only).  The work items are slices of tiles: item u of slices * tiles is slice u / tiles of a tile,
// tiles taken in super-rows of 8 tile rows (column by column inside), and round j of the grid deals each XCD 32
// consecutive items, which share their operand tiles as a block of 8 x 4 does.  With one slice the launch is an
// ordinary product in the order of the others.
template <int PRODUCT, bool QUAD>
__global__ __launch_bounds__(kGemmThreads) void gemm_kernel(const GemmArgs g)
{
    extern __shared__ __align__(16) char lds[];
    constexpr bool LSE = PRODUCT == kGemmLse || PRODUCT == kGemmLseStore, SPLIT = PRODUCT == kGemmSplitRows || PRODUCT == kGemmSplitPanels;
    static_assert(LSE || QUAD, "slices are whole groups of ring stages");
    constexpr int kLoads = 4;  // direct loads per wavefront and stage: two of A, two of B
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave & 1, wn = wave >> 1;  // row half (128 rows), column quarter (64 columns) of the tile
    const int xcd = (int)(blockIdx.x % (unsigned)g.nxcd), slot = (int)(blockIdx.x / (unsigned)g.nxcd);
    int64_t M = g.M, N = g.N, K = g.K;
    if (g.dyn_dim != kDynNone) {  // an extent that only the device knows (uniform: one scalar load)
        const int64_t v = dyn_extent(g.dyn, 0);
        if (g.dyn_dim == kDynM) M = v;
        else if (g.dyn_dim == kDynN) N = v;
        else K = (v + 127) / 128 * 128;
        if (v <= 0) return;
    }
    GemmCut cut;  // (part 1: LSE only)
    if constexpr (LSE) {  // (the search costs some 3 us here: done on the host where N is known there)
        if (g.dyn_dim == kDynNone) cut = g.cut;
        else cut = gemm_cut(M, N, g.nxcd, g.per_xcd, g.room);
    } else cut = gemm_plain_cut(gemm_shape(M, N, g.nxcd, g.per_xcd));
    const int ntiles = LSE ? cut.tiles0 + cut.part[1].ntiles : cut.tiles0, mtiles = cut.part[0].mtiles;
    const int nl0 = slot % cut.part[0].ncol, ml0 = slot / cut.part[0].ncol;  // (ml >= the part's ml: no place in its blocks)
    const int nl1 = LSE ? slot % cut.part[1].ncol : 0, ml1 = LSE ? slot / cut.part[1].ncol : 0;
    const int64_t tiles = (int64_t)mtiles * ntiles;
    const int slices = SPLIT ? gemm_slices(tiles, K / (kDmaK * kDmaStages), g.nxcd * g.per_xcd, g.split_max) : 1;
    const bool flat = SPLIT && slices > 1;
    const bool placed = ml0 < cut.part[0].ml || (LSE && ml1 < cut.part[1].ml);
    const int64_t p_end = uniform64(flat ? tiles * slices : placed ? (int64_t)(xcd + 1) * cut.pairs / g.nxcd : 0);
    const int nstages = (int)(K / kDmaK);
    const int wave_s = __builtin_amdgcn_readfirstlane(wave);  // the wavefront number in a scalar register

    // A work item: number p, and for a pair its column group, round and part (counted on, not divided out of p).
    struct Work {
        int64_t p;
        int grp, rnd;
        bool two;
    };
    // this workgroup's tile of a pair (its place in the block may have none: past the end of the grid or of the part)
    auto row_tile = [&](const Work &w) { return w.rnd * (LSE && w.two ? cut.part[1].ml : cut.part[0].ml) + (LSE && w.two ? ml1 : ml0); };
    auto column_tile = [&](const Work &w) {
        return LSE && w.two ? cut.tiles0 + w.grp * cut.part[1].ncol + nl1 : w.grp * cut.part[0].ncol + nl0;
    };
    auto exists = [&](const Work &w) {
        const bool two = LSE && w.two;
        return (two ? ml1 < cut.part[1].ml : ml0 < cut.part[0].ml) && row_tile(w) < mtiles && column_tile(w) < (two ? ntiles : cut.tiles0);
    };
    auto step = [&](Work &w) {
        ++w.p;
        if (++w.rnd < (LSE && w.two ? cut.part[1].rounds : cut.part[0].rounds)) return;
        w.rnd = 0;
        ++w.grp;
        if (LSE && w.p == cut.pairs0) {
            w.two = true;
            w.grp = 0;
        }
    };
    // the first work item from w on for this workgroup (p >= p_end if there is none): the next pair in this XCD's range whose
    // tile exists, or (flat) w itself
    auto seek = [&](Work w) {
        while (!flat && w.p < p_end && !exists(w)) step(w);
        return w;
    };
    auto start = [&](int64_t p) {
        Work w;
        w.p = p;
        w.two = LSE && p >= cut.pairs0;
        const int64_t q = w.two ? p - cut.pairs0 : p;
        const int rounds = w.two ? cut.part[1].rounds : cut.part[0].rounds;
        w.grp = __builtin_amdgcn_readfirstlane((int)(q / rounds));
        w.rnd = __builtin_amdgcn_readfirstlane((int)(q % rounds));
        return seek(w);
    };
    auto next_item = [&](Work w) {
        if (flat) {
            w.p += (int64_t)g.nxcd * g.per_xcd;
            return seek(w);
        }
        step(w);
        return seek(w);
    };
    // tile coordinates and stage range of a work item
    struct Item {
        int mt, nt, slice, s0, s1;
    };
    auto locate = [&](const Work &w) {
        Item it;
        it.slice = 0;
        it.s0 = 0;
        it.s1 = nstages;
        if (flat) {  // (few items: 32-bit arithmetic)
            const uint32_t u = (uint32_t)w.p, nt = (uint32_t)tiles, quads = (uint32_t)nstages / kDmaStages;
            const uint32_t slice = u / nt, tile = u % nt, super = 8u * (uint32_t)ntiles;
            it.slice = (int)slice;
            it.s0 = (int)(slice * quads / (uint32_t)slices) * kDmaStages;
            it.s1 = (int)((slice + 1) * quads / (uint32_t)slices) * kDmaStages;
            const uint32_t srow = tile / super, in = tile % super, h = min(8u, (uint32_t)mtiles - srow * 8u);
            it.mt = (int)(srow * 8u + in % h);
            it.nt = (int)(in / h);
        } else {
            it.mt = row_tile(w);
            it.nt = column_tile(w);
        }
        if constexpr (SPLIT) {  // (the divisions are done in vector registers: back to scalar ones, as what they are for)
            it.mt = __builtin_amdgcn_readfirstlane(it.mt);
            it.nt = __builtin_amdgcn_readfirstlane(it.nt);
            it.slice = __builtin_amdgcn_readfirstlane(it.slice);
            it.s0 = __builtin_amdgcn_readfirstlane(it.s0);
            it.s1 = __builtin_amdgcn_readfirstlane(it.s1);
        }
        return it;
    };

    Operand<LSE ? kRows : kPanels> opa;
    Operand<LSE ? kRows : PRODUCT == kGemmSplitRows ? kSlowRows : kPanels> opb;
    opa.init(g.A, g.lda, M, g.k_rows, wave_s, lane);
    opb.init(g.B, g.ldb, N, g.k_rows, wave_s, lane);
    const uint32_t fa_base = opa.lane_base(wm * 8), fb_base = kDmaOperandBytes + opb.lane_base(wn * 4);
    auto frag_a = [&](char *stage, int t) { return opa.fragment(stage, fa_base, t); };
    auto frag_b = [&](char *stage, int t) { return opb.fragment(stage, fb_base, t); };

    Work w_cur = start(flat ? uniform64((int64_t)xcd * g.per_xcd + slot) : uniform64((int64_t)xcd * cut.pairs / g.nxcd));
    if (w_cur.p >= p_end) return;  // uniform over the workgroup

    // The refill cursor names the tile (r_w) and stage (r_k; QUAD: the first of a group of kDmaStages stages) that
    // the next refill loads.  Past the workgroup's last tile it stays on that tile's last stage (group): reloads of
    // bytes that are already there, which keep the number of loads per stage, and with it the s_waitcnt
    // arithmetic, constant.  Rows past the end of an operand are clamped (computed, never written).
    Work r_w = w_cur;
    int r_k = 0, r_end = 0;
    auto set_tile = [&](const Work &w) {
        const Item it = locate(w);
        r_k = it.s0;
        r_end = it.s1;
        opa.set_tile(it.mt);
        opb.set_tile(it.nt);
    };
    set_tile(r_w);
    // direct load number q of one operand (0: A, 1: B) of stage r_k + u into ring slot sl
    auto refill = [&](int sl, int q, int u, int operand) {
        char *dst = lds + sl * kDmaStageBytes;
        if (operand == 0) opa.refill(dst, q, (uint32_t)(r_k + u));
        else opb.refill(dst + kDmaOperandBytes, q, (uint32_t)(r_k + u));
    };
    auto advance = [&](int step) {
        if (r_k + step < r_end) {
            r_k += step;
        } else {
            const Work next = next_item(r_w);
            if (next.p < p_end) {
                r_w = next;
                set_tile(next);
            }
        }
    };

    // prologue: fill the whole ring, then wait for the first stage and read its fragments
#pragma unroll
    for (int st = 0; st < kDmaStages; ++st) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            refill(st, q, QUAD ? st : 0, 0);
            refill(st, q, QUAD ? st : 0, 1);
        }
        if (!QUAD) advance(1);
    }
    if (QUAD) advance(kDmaStages);
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(kLoads * (kDmaStages - 1), kNoLgkmWait));  // everything issued after the first stage may fly
    __builtin_amdgcn_s_barrier();  // bare, as in the K loop: the rest of the ring stays in flight
    bf16x8_t fa[8], fb[2][4];
#pragma unroll
    for (int a = 0; a < 8; ++a) fa[a] = frag_a(lds, a);
#pragma unroll
    for (int b = 0; b < 4; ++b) fb[0][b] = frag_b(lds, b);
    int sl_dyn = 0;  // ring slot of the stage being computed (tracked only when !QUAD)

    float run_m[4], run_s[4];  // kGemmLse*: this lane's four columns over the sweep
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        run_m[b] = kNegFloor;
        run_s[b] = 0.0f;
    }

    while (w_cur.p < p_end) {
        const Item cur = locate(w_cur);
        const int64_t m0 = (int64_t)cur.mt * kGemmTile, n0 = (int64_t)cur.nt * kGemmTile;
        f32x4_t acc[8][4];
#pragma unroll
        for (int a = 0; a < 8; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[a][b][i] = 0.0f;

        // One stage out of the row fragments fa and the column fragments fb[p] (read from ring slot sl during the
        // stage before); u: the stage's position in the cursor's group (0 when !QUAD).
        auto stage = [&](const int sl, const int u, const int p) __attribute__((always_inline)) {
            const int nsl = sl + 1 == kDmaStages ? 0 : sl + 1;
            char *nxt = lds + nsl * kDmaStageBytes;
            __builtin_amdgcn_sched_barrier(0);
            // The next stage has landed (own loads: the kDmaStages - 2 stages after it may still be in flight) and
            // this stage is in registers (own reads, lgkmcnt(0)): meet.  A bare barrier: the fence that
            // __syncthreads() carries makes the compiler drain every direct load it can see in flight
            // (vmcnt(0)), which would empty the ring at each stage.
            __builtin_amdgcn_s_waitcnt(waitcnt_imm(kLoads * (kDmaStages - 2), 0));
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int a = 0; a < 8; ++a) {
                // a column fragment of the next stage, a direct load into the slot this stage came from ...
                if (a < 4) fb[p ^ 1][a] = frag_b(nxt, a);
                if ((a & 1) == 0) refill(sl, a >> 2, u, (a >> 1) & 1);
                // ... four MFMAs ...
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[a], fb[p][b], acc[a][b], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                // ... and this row fragment's successor, into the registers those MFMAs have just read
                fa[a] = frag_a(nxt, a);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        if (QUAD) {
            static_assert(kDmaStages == 4, "the unrolled loop names the four ring slots");
#pragma unroll 1
            for (int i = cur.s0; i < cur.s1; i += kDmaStages) {
                stage(0, 0, 0);
                stage(1, 1, 1);
                stage(2, 2, 0);
                stage(3, 3, 1);
                advance(kDmaStages);
            }
        } else {
#pragma unroll 1
            for (int i = 0; i < nstages; i += 2) {  // K % 64 == 0: an even number of stages
                stage(sl_dyn, 0, 0);
                advance(1);
                sl_dyn = sl_dyn + 1 == kDmaStages ? 0 : sl_dyn + 1;
                stage(sl_dyn, 0, 1);
                advance(1);
                sl_dyn = sl_dyn + 1 == kDmaStages ? 0 : sl_dyn + 1;
            }
        }

        // ---- the tile's epilogue, while the next tile's first stages arrive ----
        const Work w_next = next_item(w_cur);
        const bool edge = m0 + kGemmTile > M || n0 + kGemmTile > N;  // uniform
        if constexpr (SPLIT) {
            float *stage_tile = reinterpret_cast<float *>(lds + kDmaRingBytes + kGemmRedBytes + wave_s * kStageBytes);
            // (a copy of the lane number that the compiler cannot see through: the four stores' addresses are computed
            // here instead of being kept, and spilled, across the K loop)
            int lane_e = lane;
            asm volatile("" : "+v"(lane_e));
            if (flat) {  // this slice's fp32 contribution, added up by gemm_split_reduce_kernel
                float *part = g.split + (int64_t)cur.slice * M * N;
                if (edge) store_tile_edge<F32>(acc, part, N, m0, n0, M, N, wm, wn, lane_e);
                else store_tile_wide<F32>(acc, part, N, m0, n0, wm, wn, lane_e, stage_tile);
            } else {
                if (edge) store_tile_edge<Bf16>(acc, g.C, g.ldc, m0, n0, M, N, wm, wn, lane_e);
                else store_tile_wide<Bf16>(acc, g.C, g.ldc, m0, n0, wm, wn, lane_e, stage_tile);
            }
        } else if constexpr (PRODUCT != kGemmLse) {
            char *stage_tile = lds + kDmaRingBytes + kGemmRedBytes + wave_s * kStageBytes;
            int lane_e = lane;  // (as above)
            asm volatile("" : "+v"(lane_e));
            using DT = typename std::conditional<PRODUCT == kGemmPanelsBf16, Bf16, F32>::type;
            if (PRODUCT == kGemmPanelsF32 && g.accumulate != 0)
                add_tile_transposed(acc, reinterpret_cast<float *>(g.C), g.ldc, m0, n0, M, N, wm, wn, lane_e);
            else if (edge) store_tile_lines<DT, true>(acc, g.C, g.ldc, m0, n0, M, N, wm, wn, lane_e, stage_tile);
            else store_tile_lines<DT, false>(acc, g.C, g.ldc, m0, n0, M, N, wm, wn, lane_e, stage_tile);
        }
        if constexpr (LSE) {
            const bool ragged = m0 + kGemmTile > M;
            const int mlim = (int)(M - m0) - wm * 128 - (lane >> 4) * 4;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                if (ragged) fold_column<true>(acc, b, mlim, run_m[b], run_s[b]);
                else fold_column<false>(acc, b, mlim, run_m[b], run_s[b]);
                __builtin_amdgcn_sched_barrier(0);
            }
            // end of this column group's sweep: merge the four lane groups, then the two row halves, and write the
            // workgroup's partial of its 256 columns (the reduction has LDS of its own: the ring keeps running)
            if (w_next.p >= p_end || column_tile(w_next) != cur.nt) {
                float2 *red = reinterpret_cast<float2 *>(lds + kDmaRingBytes);  // [2][256]
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    MaxSum mine = {run_m[b], run_s[b]};
#pragma unroll
                    for (int off = 16; off <= 32; off <<= 1) {
                        const MaxSum other = {__shfl_xor(mine.m, off, kWave), __shfl_xor(mine.s, off, kWave)};
                        mine = combine(mine, other);
                    }
                    if (lane < 16) lds_put(red + wm * kGemmTile + wn * 64 + b * 16 + lane, f32x2_t{mine.m, mine.s});
                    run_m[b] = kNegFloor;
                    run_s[b] = 0.0f;
                }
                // (the empty asm statements keep the compiler from moving LDS accesses across the bare barriers)
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_waitcnt(waitcnt_imm(kNoVmWait, 0));
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                if (tid < kGemmTile) {
                    const f32x2_t q0 = lds_get<f32x2_t>(red + tid);
                    const f32x2_t q1 = lds_get<f32x2_t>(red + kGemmTile + tid);
                    const MaxSum tot = combine(MaxSum{q0[0], q0[1]}, MaxSum{q1[0], q1[1]});
                    const int64_t c0 = min((int64_t)cut.tiles0 * kGemmTile, N);  // columns of part 0
                    const bool two = n0 >= c0;
                    float2 *partial = g.partial + (two ? (int64_t)g.nxcd * cut.part[0].ml * c0 + (xcd * cut.part[1].ml + ml1) * (N - c0) - c0
                                                       : (xcd * cut.part[0].ml + ml0) * c0);
                    if (n0 + tid < N) partial[n0 + tid] = make_float2(tot.m, tot.s);
                }
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_waitcnt(waitcnt_imm(kNoVmWait, 0));  // red is read before anyone writes it again
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
        }
        w_cur = w_next;
    }
    // drain: the reloads past the last stage must have landed before the workgroup ends
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));
    __builtin_amdgcn_s_barrier();
}

// C (bfloat16) = the slices of a kGemmSplit* launch, added in ascending order; nothing when the launch did not slice.
// Memory bound: 8 elements per thread and step, 2 x 16 bytes per slice.
__global__ __launch_bounds__(256) void gemm_split_reduce_kernel(const GemmArgs g)
{
    const int64_t M = g.dyn_dim == kDynM ? dyn_extent(g.dyn, 0) : g.M, N = g.N;
    if (M <= 0) return;
    const int64_t tiles = ((M + kGemmTile - 1) / kGemmTile) * ((N + kGemmTile - 1) / kGemmTile);
    const int slices = gemm_slices(tiles, g.K / (kDmaK * kDmaStages), g.nxcd * g.per_xcd, g.split_max);
    if (slices <= 1) return;
    const int64_t step = (int64_t)gridDim.x * blockDim.x * 8;
    for (int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 8; i < M * N; i += step) {  // N % 8 == 0
        float f[8];
        for (int q = 0; q < slices; ++q) {
            const float4 *src = reinterpret_cast<const float4 *>(g.split + (int64_t)q * M * N + i);
            const float4 a = src[0], b = src[1];
            const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) f[e] = q ? f[e] + v[e] : v[e];
        }
        *reinterpret_cast<uint4 *>(reinterpret_cast<uint16_t *>(g.C) + (i / N) * g.ldc + i % N) = pack<Bf16>(f);
    }
}

// ---------------------------------------------------------------------------------------
// host side

// Shape of the persistent grid on the current device: one workgroup per compute unit, dealt round-robin to the
// XCDs by the dispatcher (eight XCDs on the full chip; a partition with fewer than 64 compute units is one XCD).
GemmGrid gemm_grid()
{
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
        cus = kGemmMaxBlocks;
    if (cus > kGemmMaxBlocks) cus = kGemmMaxBlocks;
    GemmGrid gg;
    gg.nxcd = (cus >= 64 && cus % 8 == 0) ? 8 : 1;
    gg.per_xcd = cus / gg.nxcd;
    return gg;
}

template <int PRODUCT, bool QUAD>
static hipError_t launch_gemm_t(const GemmArgs &g, hipStream_t s)
{
    static LdsLimitState lds_limit;
    auto *kernel = gemm_kernel<PRODUCT, QUAD>;
    const hipError_t attr_err = ensure_lds_limit(reinterpret_cast<const void *>(kernel), kGemmLdsBytes, lds_limit);
    if (attr_err != hipSuccess) return attr_err;
    hipLaunchKernelGGL(kernel, dim3(g.nxcd * g.per_xcd), dim3(kGemmThreads), kGemmLdsBytes, s, g);
    return hipGetLastError();
}

hipError_t launch_gemm(const GemmArgs &args, int product, hipStream_t s)
{
    GemmArgs g = args;
    const GemmGrid gg = gemm_grid();
    g.nxcd = gg.nxcd;
    g.per_xcd = gg.per_xcd;
    const bool lse = product == kGemmLse || product == kGemmLseStore, quad = g.K % (kDmaK * kDmaStages) == 0;
    const bool panels = product == kGemmPanelsBf16 || product == kGemmPanelsF32;
    if (lse && (!g.partial || g.room < (int64_t)gemm_partial_entries(g.N))) return hipErrorInvalidValue;
    if (lse && g.dyn_dim == kDynNone) g.cut = gemm_cut(g.M, g.N, g.nxcd, g.per_xcd, g.room);
    // what the kernel's 32-bit offsets and its stage arithmetic assume
    if (g.M <= 0 || g.N <= 0 || g.K <= 0 || g.K % 64 != 0 || g.lda % 8 != 0 || g.ldb % 8 != 0 || g.lda > (1 << 22) ||
        g.ldb > (1 << 22))
        return hipErrorInvalidValue;
    if (g.dyn_dim != kDynNone && !g.dyn.n) return hipErrorInvalidValue;
    if (g.dyn_dim == kDynK && !panels) return hipErrorInvalidValue;
    if (product != kGemmLse && (g.ldc % 8 != 0 || (reinterpret_cast<uintptr_t>(g.C) & 15) != 0)) return hipErrorInvalidValue;
    // C^T: 16-byte stores along M
    if ((product == kGemmLseStore || panels) && (g.M % (product == kGemmPanelsBf16 ? 8 : 4) != 0 || g.dyn_dim == kDynM))
        return hipErrorInvalidValue;
    if (lse) {
        if (g.lda < g.K || g.ldb < g.K) return hipErrorInvalidValue;
        if (product == kGemmLse) return quad ? launch_gemm_t<kGemmLse, true>(g, s) : launch_gemm_t<kGemmLse, false>(g, s);
        return quad ? launch_gemm_t<kGemmLseStore, true>(g, s) : launch_gemm_t<kGemmLseStore, false>(g, s);
    }
    if (!quad || g.lda % 64 != 0 || g.lda < g.K) return hipErrorInvalidValue;
    if (panels) {
        if (g.ldb % 64 != 0 || g.ldb < g.K) return hipErrorInvalidValue;
        return product == kGemmPanelsBf16 ? launch_gemm_t<kGemmPanelsBf16, true>(g, s) : launch_gemm_t<kGemmPanelsF32, true>(g, s);
    }
    if (g.N % 64 != 0 || g.dyn_dim == kDynN || (g.split_max > 1 && !g.split)) return hipErrorInvalidValue;
    hipError_t e = hipErrorInvalidValue;
    if (product == kGemmSplitRows && g.k_rows > 0 && g.ldb >= g.N) e = launch_gemm_t<kGemmSplitRows, true>(g, s);
    else if (product == kGemmSplitPanels && g.ldb % 64 == 0 && g.ldb >= g.K) e = launch_gemm_t<kGemmSplitPanels, true>(g, s);
    if (e != hipSuccess || g.split_max <= 1) return e;
    hipLaunchKernelGGL(gemm_split_reduce_kernel, dim3(4 * g.nxcd * g.per_xcd), dim3(256), 0, s, g);
    return hipGetLastError();
}

}  // namespace a3po
