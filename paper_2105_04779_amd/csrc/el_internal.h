// Internal declarations shared by the library's translation units (not installed).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include "el_attn.h"

namespace el {

// ---- storage element types --------------------------------------------------------------
struct bf16_t { uint16_t bits; };
typedef _Float16 f16_t;

__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(f16_t v) { return (float)v; }
__device__ __forceinline__ float to_f32(bf16_t v) { return __uint_as_float(((uint32_t)v.bits) << 16); }

// round-to-nearest-even conversions for stores in the storage dtype
__device__ __forceinline__ void from_f32(float x, float *p) { *p = x; }
__device__ __forceinline__ void from_f32(float x, f16_t *p) { *p = (f16_t)x; }
__device__ __forceinline__ void from_f32(float x, bf16_t *p) {
    uint32_t u = __float_as_uint(x);
    if ((u & 0x7fffffffu) > 0x7f800000u) { p->bits = 0x7fc0; return; }
    u += 0x7fffu + ((u >> 16) & 1u);
    p->bits = (uint16_t)(u >> 16);
}

// x = high + low, both in the 16-bit storage type (the pair carries ~16 mantissa bits of x)
template <bool BF16>
__device__ __forceinline__ void split16(float x, uint16_t &hi, uint16_t &lo)
{
    if (BF16) {
        bf16_t h, l2;
        from_f32(x, &h);
        from_f32(x - to_f32(h), &l2);
        hi = h.bits; lo = l2.bits;
    } else {
        const f16_t h = (f16_t)x, l2 = (f16_t)(x - (float)h);
        hi = __builtin_bit_cast(uint16_t, h); lo = __builtin_bit_cast(uint16_t, l2);
    }
}

// ---- LDS staging helpers of the attention core ---------------------------------------------
// One 1 KB piece of a row, fetched by one wavefront straight into LDS.  `lds_addr` is the
// LDS byte address the piece starts at (lane i lands at +16 i), `voff` the lane's byte offset from
// the wave-uniform global base.  Issued through inline assembly so that the compiler does not
// serialise later LDS reads of the *other* tile buffer behind it; completion is awaited
// explicitly (s_waitcnt vmcnt(0)) before the barrier that publishes the tile.
__device__ __forceinline__ void dma_piece(unsigned lds_addr, unsigned voff, const char *sbase)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds_addr), "v"(voff), "s"(sbase) : "memory", "m0");
}
__device__ __forceinline__ void dma_row_2k(unsigned lds_addr, unsigned voff, const char *sbase)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2\n\tglobal_load_lds_dwordx4 %1, %2 offset:1024"
                 :: "s"(lds_addr), "v"(voff), "s"(sbase) : "memory", "m0");
}

// The same requests with the non-temporal hint: the lines are not kept in L2 or in the memory-side cache.
// For a stream far larger than that cache this leaves it to the data that IS re-read (weights, expanded
// queries, partial results) and raises the streaming rate itself.
__device__ __forceinline__ void dma_piece_nt(unsigned lds_addr, unsigned voff, const char *sbase)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                 :: "s"(lds_addr), "v"(voff), "s"(sbase) : "memory", "m0");
}
__device__ __forceinline__ void dma_row_2k_nt(unsigned lds_addr, unsigned voff, const char *sbase)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt\n\tglobal_load_lds_dwordx4 %1, %2 offset:1024 nt"
                 :: "s"(lds_addr), "v"(voff), "s"(sbase) : "memory", "m0");
}

static inline size_t dtype_size(int dt) { return dt == EL_F32 ? 4 : 2; }
static inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// EL-Q for the MFMA core is stored in the order its score wavefronts load it: 1 KB fragments of 16 rows x 32
// columns (row-major inside: element (r16, c32) at r16 * 32 + c32), ordered [batch element][row / 16][column / 32]
// [plane: 0 high, 1 low], so that one load instruction of a wavefront (lane = 4 r16 + column group) reads one
// contiguous fragment.  Returns the element index of (b, row, col) of a plane; Rs = padded row count, a multiple
// of 16.
__host__ __device__ __forceinline__ size_t elq_frag_index(int b, int row, int col, int plane, int Rs, int d_m)
{
    const size_t frag = (((size_t)b * (Rs >> 4) + (row >> 4)) * (d_m >> 5) + (col >> 5)) * 2 + plane;
    return frag * 512 + (size_t)(row & 15) * 32 + (col & 31);
}

// Row-major 16-bit matrices [rows, K] that a 16x16x32 MFMA reads as 16-row operands are kept in its fragment order too
// (the pieces X of the core, the head outputs A): 1 KB fragments of 16 rows x 32 columns, [row / 16][column / 32], so
// that an operand load of a wavefront is contiguous instead of 16 segments of 64 bytes.  Rows are padded to 16.
__host__ __device__ __forceinline__ size_t frag16_index(int row, int col, int K)
{
    return ((size_t)(row >> 4) * (K >> 5) + (col >> 5)) * 512 + (size_t)(row & 15) * 32 + (col & 31);
}

// ---- compile-time limits -----------------------------------------------------------------
constexpr int kMaxParts = 15;       // pieces (fp16) per batch element the workspace of the MFMA core has room for
constexpr int kMaxPartsGeneric = 8; // key-range partials (fp32) of the generic core
constexpr int kGenericMaxDm = 8192; // widest d_model the generic core kernel covers
constexpr int kScanMax = 1024;      // most batch elements whose tiles the streaming core cuts as one list
constexpr int kSpanMax = 1024;      // most spans of that list
constexpr int kShortTiles = 4;      // tiles that a workgroup of the core of short spans holds in LDS (its wide ones: up to 8, see plan_wide_spans)

// Where the partial results ("pieces") of batch element b live: `np` consecutive slots from `slot0` in the partial
// buffers Xp [slot, Rs, d_m] and ML [slot, Rs, 2].  Generic core: every element has `parts` of them.  MFMA core: looked
// up in the table of the cut (cut.h).
struct PieceMap {
    const int2 *table;      // [B] (first slot, pieces); null: slots b * parts ..
    int parts;
};
__device__ __forceinline__ void piece_range(const PieceMap &m, int b, int &slot0, int &np)
{
    if (!m.table) { slot0 = b * m.parts; np = m.parts; return; }
    const int2 e = m.table[b];
    slot0 = e.x; np = e.y;
}

// What build_cut (cut.h) needs to know
struct CutArgs {
    const int32_t *lengths;
    int4 *spans;            // [G][2]: (element, tile of it, tiles, first slot), (lengths of the first four elements)
    int2 *pieces;           // [B] (first slot, pieces)
    int n, B, G, kcost;
    int short_tiles;        // nonzero: per element, into spans of at most so many tiles (G is enough of them)
};

// ---- problem description handed to the launchers ------------------------------------------
struct Problem {
    int B, beam, n, heads, d_m, d_k, hd, R;
    int dtype, out_dtype;
    const void *H;
    int64_t H_batch_stride;
    const int32_t *lengths;
    const void *queries;
    void *out;
};

// Workspace carve-up (device pointers into the caller's buffer).
struct Workspace {
    float *Qp;      // [B*beam, hd]                 a1 result: fp32 (generic) or fp16 (MFMA GEMMs), scaled
    void *ELQ;      // [B, Rpad, d_m]               fp32 (generic) or fp16 (MFMA core)
    float *Xp;      // [B, parts, Rpad, d_m]        partial weighted sums: fp16 in fragment order (MFMA), fp32 (generic)
    float *ML;      // [B, parts, Rpad, 2]          running max and sum of each partial
    float *Xn;      // [B, R, d_m]                  merged, normalised weighted sums (generic path)
    float *A;       // [B*beam, hd]                 a6 result: fp32 (generic) or fp16 in fragment order (MFMA projections)
    int4 *spans;    // [slots][2]                   the cut of the MFMA core (see CutArgs)
    int2 *pieces;   // [B]
    int slots;      // pieces Xp and ML have room for (batch elements the workspace was laid out for x kMaxParts)
};

struct Weights {    // library-owned copies; every product reads both operands along the contraction, hence the transposes
    void *WqT, *Wk, *bq;            // (W^Q)^T and W^K as it is (a head's slice of a row is the contraction), storage dtype
    void *WqP, *WkP, *WvP, *WoP;    // MFMA projections: all four in fragments; W^Q in the storage type, the others in fp16
    void *WvTs, *WoTs;              // fp32-arithmetic projections: (W^V)^T, (W^O)^T in the storage dtype
    float *c_out;                   // [d_m] = b_o + b_v . W_o, fp32
    float *bk32, *bv32, *bo32;      // [h*d_k], [h*d_k], [d_m] in fp32 (zeros when absent): only the segment form reads them
};

} // namespace el

// The context behind the opaque handle.
struct el_attn_ctx {
    el_attn_config cfg;
    int hd;                 // heads * d_k
    int Rpad_max;           // max_beam*heads rounded up to a multiple of 64
    el::Weights w;
    void *ws_base;
    size_t ws_bytes;        // bound size
    size_t ws_need;         // required size
    int splits_override;    // 0 = automatic
    int nrg_override;       // 0 = automatic
    int use_mfma_core;      // MFMA attention core available for this (dtype, d_m)
    int use_mfma_gemm;      // MFMA projection GEMMs available for this (dtype, d_m, d_k)
    int device;
    int num_cus;            // compute units of that device
    // optional event pairs around the core kernel (measurement aid)
    hipEvent_t *ev;         // 2 * ev_cap events, or null
    int ev_cap, ev_used;
};

namespace el {

// generic (fp32 arithmetic) kernels -- generic_kernels.hip
hipError_t launch_cout(const el_attn_ctx *ctx, const void *WoT, const void *bv, const void *bo, hipStream_t s);   // WoT in the storage dtype
hipError_t launch_qproj_generic(const el_attn_ctx *ctx, const Problem &p, const Workspace &ws, hipStream_t s);
hipError_t launch_elq_generic(const el_attn_ctx *ctx, const Problem &p, const float *Qp, float *elq, hipStream_t s);
bool scores_fit(const Problem &p);                    // the core through scores in memory applies; the next two are for the rest
hipError_t launch_core_scores(const el_attn_ctx *ctx, const Problem &p, const Workspace &ws, hipStream_t s);
hipError_t launch_core_generic(const el_attn_ctx *ctx, const Problem &p, const Workspace &ws, int parts, hipStream_t s);
hipError_t launch_merge_generic(const el_attn_ctx *ctx, const Problem &p, const Workspace &ws, int parts, int Rstride, hipStream_t s);
hipError_t launch_vproj_generic(const el_attn_ctx *ctx, const Problem &p, const Workspace &ws, hipStream_t s);
hipError_t launch_oproj_generic(const el_attn_ctx *ctx, const Problem &p, const Workspace &ws, const float *bias32, hipStream_t s);
hipError_t launch_vec_f32(int dtype, const void *src, float *dst, int n, hipStream_t s);
// the whole step of a narrow layer in one launch -- small_step.hip
bool small_step_applies(const Problem &p);
hipError_t launch_small_step(const el_attn_ctx *ctx, const Problem &p, hipStream_t s);
// segment form (decoder-only models): statistics + biased head outputs of one segment; merge of several
struct SegFinishArgs {
    const float *A;           // [rows, hd]: the segment's normalised head outputs without b^V
    const float *Qp;          // [rows, hd]: projected queries as a1 left them (scaled by 1/sqrt(d_k))
    const float *ML;          // [slot, Rstride, 2] statistics of the pieces (see PieceMap)
    PieceMap pm;
    const float *bk32, *bv32;
    float *seg_A, *seg_lse;
    int beam, heads, d_k, hd, Rstride;
    float ml_to_nat;          // factor that turns ML's maxima into natural-log units
};
struct SegOut { float *A, *lse; };   // a segment's results
constexpr int kMaxSegments = 4;
struct SegMergeArgs {
    const float *A[kMaxSegments];
    const float *lse[kMaxSegments];
    void *A_out;              // [rows, hd] fp16 (in fragment order) or fp32
    int nseg, heads, d_k, hd;
};
hipError_t launch_seg_finish(const SegFinishArgs &a, int rows, hipStream_t s);     // around the fp32-arithmetic projections
hipError_t launch_seg_merge(const SegMergeArgs &a, bool out_f16, int rows, hipStream_t s);

// MFMA attention core -- core_stream.hip (the kernel), core_mfma.hip (planning, launch, helpers)
struct CorePlan {
    int nrg;      // 16-row groups per workgroup (1 or 2)
    int block_groups;   // 16-row groups of the row blocks the spans are planned for: nrg, or 2 where two workgroups of the streaming core share one
    int nblocks;  // row blocks (workgroups sharing one H range)
    int Rs;       // padded row count of ELQ / partial buffers = nblocks * 16 * nrg
    int G;        // spans the tiles of all elements are cut into (more than kScanMax elements: one span each)
    int kcost;    // what crossing into a new element costs a workgroup, in tiles (see cut.h)
    int short_tiles;    // nonzero: every element is cut into spans of at most this many tiles, for the core of short spans
};
// Arguments of the streaming core (core_stream.hip)
struct StreamArgs {
    const void *H;
    int64_t h_stride;        // elements between batch elements
    const int32_t *lengths;
    const uint16_t *elq;     // EL-Q as high + low 16-bit planes in the storage type, scaled by log2(e)/sqrt(d_k),
                             //   in fragment order (see elq_frag_index)
    f16_t *Xp;               // [slot, Rs, DM] fp16, each piece already divided by its own sum, in fragment order (frag16_index)
    float *ML;               // [slot, Rs, 2]  (reference max in log2 units, sum)
    const int4 *spans;       // the cut (see CutArgs)
    const void *next_w[2];   // packed weights of a6 and a7, read ahead for them (null: not those projections)
    int n, B, R, Rs, nblocks, G, num_cus;
    int stream_hint;         // nonzero: fetch H with the non-temporal hint (H far larger than the memory-side cache)
};
// A workgroup of either core on a compute unit that the spans leave idle: pulls the weights of a6 and a7 towards this XCD's L2,
// one dword of every 128-byte line, an eighth of either matrix per XCD (the projections deal their column blocks that way).
template <int DM>
__device__ __forceinline__ void read_ahead(const StreamArgs &a, int per_xcd)
{
    constexpr int LINES = DM * DM * 2 / 8 / 128;
    for (int t = ((blockIdx.x >> 3) - per_xcd) * 512 + threadIdx.x; t < 2 * LINES; t += (gridDim.x / 8 - per_xcd) * 512) {
        const char *src = (const char *)a.next_w[t >= LINES] + ((size_t)(blockIdx.x & 7) * LINES + (t >= LINES ? t - LINES : t)) * 128;
        const int v = *(const volatile int *)src;
        asm volatile("" :: "v"(v));
    }
}
// Workgroups of a core.  Where at least a quarter of the compute units is idle, 64 more read the weights of a6 and a7 ahead: a
// decoder's layers come with weights of their own, cold at every step.  Twelve layers, 4 sentences, d_m 1024: streaming core 320 ->
// 311.4 us, core of short spans 284.3 -> 277.2; one sentence, one layer (its weights stay in the memory-side cache): 23.7 -> 23.4, 20.9 ->
// 20.9.  In workgroups that also stream, the same reads cost 1 us: their other requests return after them.
inline dim3 core_grid(const StreamArgs &a)
{
    dim3 grid(((a.G * a.nblocks + 7) / 8) * 8);
    if (a.next_w[0] && (int)grid.x + 64 <= a.num_cus) grid.x += 64;
    return grid;
}
hipError_t launch_core_short(const StreamArgs &a, int d_m, bool bf16, int tiles, int rg, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1);   // core_short.hip
hipError_t launch_core_stream(const StreamArgs &a, int d_m, bool bf16, int rg, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1);
bool core_mfma_supported(int dtype, int d_m);
// what a step launches: the streaming core or, where neither override is set and it is the faster one, the core of short spans
// (wide: the wide workgroups of the core of short spans are allowed, as they are in a step; el_attn_plan_preview and
// el_attn_plan_short_core ask without them, el_attn_plan_step with them)
CorePlan plan_core_mfma(const Problem &p, int splits_override, int nrg_override, int num_cus, int max_slots, bool wide);
CutArgs cut_args(const Problem &p, const CorePlan &pl, const Workspace &ws);
PieceMap piece_map(const Workspace &ws);
hipError_t launch_cut(const CutArgs &c, hipStream_t s);      // the cut on its own, for a core that k_qelq does not precede
hipError_t launch_elq_f16(const el_attn_ctx *ctx, const Problem &p, const Workspace &ws, const CorePlan &pl, hipStream_t s);
hipError_t launch_core_mfma(const el_attn_ctx *ctx, const Problem &p, const Workspace &ws, const CorePlan &pl, hipStream_t s,
                            hipEvent_t ev0, hipEvent_t ev1);   // events, if given, bracket the kernel itself
hipError_t launch_merge_exp2(const el_attn_ctx *ctx, const Problem &p, const Workspace &ws, const CorePlan &pl, hipStream_t s);

// MFMA projection GEMMs -- gemm_mfma.hip
bool gemm_mfma_supported(int dtype, int d_m, int d_k);
hipError_t launch_transpose(size_t elem, const void *src, void *dst, int rows, int cols, hipStream_t s);
enum PackKind { kPackWq, kPackWk, kPackWv, kPackWo };
hipError_t launch_pack(int dtype, PackKind kind, const void *W, void *P, int d_m, hipStream_t s);
hipError_t launch_qelq_mfma(const el_attn_ctx *ctx, const Problem &p, const Workspace &ws, const CorePlan &pl, float scale, bool keep_qp, hipStream_t s);   // builds the cut as well
hipError_t launch_vproj_mfma(const el_attn_ctx *ctx, const Problem &p, const Workspace &ws, const CorePlan &pl, const SegOut *seg, hipStream_t s);   // seg: the segment form
hipError_t launch_oproj_mfma(const el_attn_ctx *ctx, const Problem &p, const Workspace &ws, const float *bias32, hipStream_t s);

} // namespace el
