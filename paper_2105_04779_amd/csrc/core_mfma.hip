// Planning and launch of the MFMA attention core (steps a3-a5 of the EL-attention decode step; the
// kernels themselves are in core_stream.hip and, for short spans, core_short.hip), plus the two small fp32-FMA kernels that stand in for the MFMA
// projections around it when the head size is not 64: the query expansion as a high + low pair of
// 16-bit planes (in the fragment order the core loads) and the log-sum-exp merge of the pieces.
#include <cmath>
#include <cstdlib>
#include "el_internal.h"
#include "cut.h"

namespace el {

// a2 for the MFMA core: EL-Q pre-multiplied by log2(e) (Qp already carries 1/sqrt(d_k)), as a high and a
// low plane in the storage type.
template <typename T, bool BF16>
__global__ void k_elq_planes(const float *__restrict__ Qp, const T *__restrict__ Wk, uint16_t *__restrict__ planes,
                             int beam, int d_m, int d_k, int hd, int R, int Rs)
{
    const int d = blockIdx.x * 256 + threadIdx.x;
    const int r = blockIdx.y, b = blockIdx.z;
    if (d >= d_m) return;
    const int i = r / beam, j = r % beam;   // Qp carries 1/sqrt(d_k) only on this path
    const float *qp = Qp + ((size_t)b * beam + j) * hd + (size_t)i * d_k;
    const T *wk = Wk + (size_t)d * hd + (size_t)i * d_k;
    float acc = 0.f;
    for (int c = 0; c < d_k; ++c) acc = fmaf(qp[c], to_f32(wk[c]), acc);
    acc *= 1.4426950408889634f;
    split16<BF16>(acc, planes[elq_frag_index(b, r, d, 0, Rs, d_m)], planes[elq_frag_index(b, r, d, 1, Rs, d_m)]);
}

// Log-sum-exp merge of normalised fp16 pieces (reference maxima in log2 units):
// X = sum_p (w_p l_p) Xhat_p / sum_p (w_p l_p),  w_p = 2^(m_p - M).
__global__ void k_merge_exp2(const f16_t *__restrict__ Xp, const float *__restrict__ ML, float *__restrict__ Xn,
                             int d_m, int R, int Rs, const PieceMap pm)
{
    const int d = blockIdx.x * 256 + threadIdx.x;
    const int r = blockIdx.y, b = blockIdx.z;
    if (d >= d_m) return;
    int slot0, np;
    piece_range(pm, b, slot0, np);
    float M = -INFINITY;
    for (int p = 0; p < np; ++p) {
        const size_t rowi = ((size_t)slot0 + p) * Rs + r;
        if (ML[rowi * 2 + 1] > 0.f) M = fmaxf(M, ML[rowi * 2]);
    }
    float num = 0.f, den = 0.f;
    for (int p = 0; p < np; ++p) {
        const size_t rowi = ((size_t)slot0 + p) * Rs + r;
        const float mp = ML[rowi * 2], lp = ML[rowi * 2 + 1];
        if (lp > 0.f) {
            const float wgt = exp2f(mp - M) * lp;
            num = fmaf(wgt, (float)Xp[((size_t)slot0 + p) * Rs * d_m + frag16_index(r, d, d_m)], num);
            den += wgt;
        }
    }
    Xn[((size_t)b * R + r) * d_m + d] = num / den;
}


// ---------------------------------------------------------------------------------------------
bool core_mfma_supported(int dtype, int d_m)
{
    return (dtype == EL_F16 || dtype == EL_BF16) && (d_m == 512 || d_m == 768 || d_m == 1024);
}

// How much the work is cut.  A workgroup takes 16 or 32 of the R = heads x beams rows that share one H (the
// row blocks of one span read the same tiles, the second one from L2) and one span of the list of all
// valid 16-row tiles.  Lengths live on the device, so the host fixes only the number of spans G: one
// workgroup per compute unit when the longest possible list gives every span at least kMinSpan tiles,
// fewer otherwise (but not fewer than one span per batch element); build_cut lays the spans over the actual lengths.
// Batches beyond kScanMax elements are not cut: one workgroup per (element, row block), scheduled by the hardware.
// What meets the line are long elements on few compute units, in a context prepared for many, and what the tuning knobs keep off the core
// of short spans.  Whole steps on this core, 8 tiles against 4 (a further piece is cheap since the merge takes several of them side by
// side; before it did, 8 was the faster one): d_m 1024, 1 beam, 16 of 960 positions 26.1 / 25.2 us, one of 6000 24.9 / 25.8, of 1024 21.5 / 19.2;
// 4 beams, one of 1000 22.5 / 20.5; d_m 512, 8 rows, 16 of 960 19.6 / 19.2, one of 6000 20.4 / 20.4.
constexpr int kMinSpan = 4;
// What moving on to the next batch element costs a workgroup, in tiles of streaming time: the expanded queries of
// the new element (128 KB for 32 rows) and the write-out of the finished piece.  Spans that cross an element hold
// that many tiles fewer, so that all workgroups finish together (measured on 64 ragged inputs of 512-1024 rows:
// workgroups with a crossing ended 5-6 us after the others).
constexpr int kBoundaryCost = 4;

// Tiles per span up to which two workgroups of 16 rows share a row block of 32, all of them on the chip at once.  Half the
// expanded queries to wait for and half the products per tile, against twice the tiles per span where the spans fill the
// chip.  Whole steps (those that do not run on the core of short spans), 32 against 16 rows: d_m 1024, 64 rows, 16 of 150 to 300
// positions 30.3 / 29.2 us, 16 of 512 (8 tiles) 32.5 / 31.2, 24 of 512 (12 tiles) 33.4 / 33.0; 32 rows, 32 of 512 34.6 / 30.3; 128 rows, 8 of
// 512 33.6 / 31.5; d_m 768, 60 rows, 16 of 256 to 512 29.1 / 26.8; 36 rows 28.3 / 26.1; d_m 512, 40 rows 22.6 / 21.1.  Of 254 such shapes of
// 24 to 128 rows 169 gain, up to 15 %, and 85 lose, up to 9 %: the 16-row workgroups of many elements fill the chip, so that their spans
// cross elements more often, and rows that fill blocks of 32 evenly have nothing to gain from blocks of 16: d_m 768, 96 rows, 24 of
// 150 to 300 29.3 / 32.1; 24 rows, 64 of 200 25.4 / 27.6; d_m 512, 32 rows, 48 of 512 23.6 / 24.9.
// The wide workgroups of the core of short spans (plan_wide_spans) have since taken most of these; what still meets this line is
// d_m 1024 between one round of those and 12 tiles, and shapes that miss their round by the padding of a last span.
constexpr int kHalfBlockTiles = 12;

static CorePlan plan_stream(const Problem &p, int splits_override, int nrg_override, int num_cus, int max_slots)
{
    CorePlan pl;
    const int tiles = (p.n + 15) / 16;
    pl.block_groups = p.R <= 16 || nrg_override == 1 ? 1 : 2;
    pl.nrg = pl.block_groups;
    pl.nblocks = (p.R + 31) / 32;
    if (nrg_override == 0 && pl.nrg == 2 && (long)p.B * tiles * pl.nblocks * 2 <= (long)kHalfBlockTiles * num_cus) pl.nrg = 1;
    pl.nblocks = (p.R + 16 * pl.nrg - 1) / (16 * pl.nrg);
    pl.Rs = pl.nblocks * 16 * pl.nrg;
    pl.kcost = kBoundaryCost;
    pl.short_tiles = 0;
    if (p.B > kScanMax) { pl.G = p.B; return pl; }
    long G;
    if (splits_override > 0) {
        G = (long)p.B * splits_override;                   // about that many pieces per element
    } else {
        const long by_cu = num_cus / pl.nblocks > 0 ? num_cus / pl.nblocks : 1;
        long by_len = (long)p.B * tiles / kMinSpan > 0 ? (long)p.B * tiles / kMinSpan : 1;
        // short inputs: a span per batch element rather than spans of kMinSpan tiles that each cross into a second
        // element and fetch its expanded queries as well (B = 64, n = 64: 16 instead of 23 us)
        const long per_elem = p.B < by_cu ? p.B : by_cu;
        if (by_len < per_elem) by_len = per_elem;
        G = by_cu < by_len ? by_cu : by_len;
    }
    if (G > max_slots - p.B) G = max_slots - p.B;
    if (G > kSpanMax) G = kSpanMax;
    if (G < 1) G = 1;
    pl.G = (int)G;
    return pl;
}

// Elements of thousands of positions (a context prepared for many, called with one to three): the streaming core's cut mostly has
// spans of five tiles, a fifth fewer pieces.  The line was drawn where a further piece cost the merge 0.3 us (177 shapes of three to
// eight more: 1.00 to 1.13 times as fast).  Since the merge takes several pieces side by side it lies on the safe side; one element, 16
// rows, streaming against short core: d_m 1024 2500 positions (8 more) 21.1 / 18.2, 5200 (17 more) 25.0 / 22.6, 7000 26.9 / 25.4, 11500 (36
// more) 32.6 / 33.1; d_m 512 17.7 / 15.7, 20.3 / 18.2, 11500 25.6 / 25.0.
constexpr int kMorePieces = 8;

// The core of short spans (core_short.hip): every element dealt out to workgroups of four tiles and 16 rows, while all of them
// run at once (spans by the longest possible element).  Beyond that a second round of workgroups waits for the first one's
// latency, which the streaming core pays once, and more pieces are written and merged.  Whole steps in bf16, the streaming core
// against the short core, elements of one length, 64 rows at d_m 1024, 48 at 768 and 32 at 512 unless it says so (us; workgroups per
// compute unit of 256):
//   d_m 1024    1 element of 613 positions 20.0 / 17.3    8 of 512 (1) 26.2 / 22.7    2 of 128 20.6 / 16.1    16 of 300 (1.25) 27.5 / 27.6
//               12 of 512 (1.5) 27.5 / 26.8    128 of 200, 16 rows (2) 34.6 / 36.3
//   d_m 768     8 of 512 (0.75) 21.8 / 17.8    16 of 300 (0.9) 23.1 / 19.1    24 of 300 (1.4) 25.5 / 25.2
//   d_m 512     24 of 300 (0.9) 19.3 / 16.5    32 of 300 (1.25) 20.2 / 18.5    64 of 300, 8 rows (1.25) 19.8 / 18.4    128 of 200, 8 rows (2) 21.8 / 19.8
// (d_m 512 has two workgroups on a compute unit and bears more than one round; 34 of 900, 16 rows (2) 21.2 / 20.8.  Most steps beyond one
// round run on the wide workgroups below.)  The line of 13 spans an element is from a merge that took one piece after another (1 beam, 17
// of 960 positions, fp16, d_m 768, 32.3 / 32.9); it lies on the safe side now: 1 beam, 16 of 960 positions d_m 1024 25.3 / 23.0, d_m 768 22.2
// / 19.9 (fp16, 17 of 960: 27.7 / 25.2, 21.9 / 20.2); 17 of 896 26.6 / 25.0, 22.1 / 19.7; 11 of 960 23.5 / 20.5, 21.7 / 18.2; 4 beams, 4 of 960
// 24.8 / 21.2.
// Where every element is one span there is no more to merge than before, and a second round pays (at d_m 512 a third):
//   d_m 1024    100 of 64 (1.6) 39.7 / 34.5    128 of 64 (2) 41.9 / 38.5    200 of 64 (3.1) 57.9 / 55.5    320 of 33 (5) 70.2 / 69.3
//   d_m 768     170 of 64 (2) 38.2 / 35.3    200 of 64 (2.3) 42.7 / 39.4    320 of 33 (3.75) 50.5 / 47.4    1000 of 64, 12 rows (3.9) 55.3 / 57.9
//   d_m 512     200 of 64 (1.6) 29.5 / 24.8    384 of 64 (3) 36.7 / 31.9    1000 of 64, 8 rows (3.9) 37.0 / 34.9
// but with one row block only up to 15/8 rounds: where both rounds are full, the streaming core has two elements on every compute
// unit and nothing idle either.  16 rows, d_m 1024: 460 of 64 49.8 / 44.1, 480 49.6 / 44.2, 512 47.2 / 46.4; 12 rows, d_m 768: 39.3 / 35.6,
// 39.4 / 36.2, 37.1 / 37.0.  Elements of a single tile gain least in a second round that is nearly empty: d_m 768, 16 positions, 89
// elements (1.04) 30.3 / 29.6 with 48 rows, 26.8 / 25.4 with 36; 44 with 96 rows 30.5 / 29.3.
static void plan_short_spans(const Problem &p, int num_cus, int max_slots, CorePlan &pl)
{
    if (p.B > kScanMax) return;
    const int per_element = (p.n + 16 * kShortTiles - 1) / (16 * kShortTiles), blocks = (p.R + 15) / 16;
    const long spans = (long)p.B * per_element;
    if (spans > kSpanMax || spans > max_slots) return;
    // eighths of a round (one row block: see above)
    const int eighths = per_element > 1 ? 8 : p.d_m == 512 ? 24 : blocks == 1 ? 15 : 16;
    if (8 * spans * blocks > (long)eighths * num_cus) return;
    if (per_element > 13) {
        if (spans > num_cus * 3 / 4) return;
        const int tiles = (p.n + 15) / 16, G = pl.G;                     // (G >= B here), tiles of a span as build_cut has them
        const int each = p.B == 1 ? (tiles + G - 1) / G : (2 * p.B * tiles + 2 * G - p.B - 1) / (2 * G - p.B);
        if (per_element - (tiles + each - 1) / each > kMorePieces) return;
    }
    pl.nrg = pl.block_groups = 1; pl.nblocks = blocks; pl.Rs = blocks * 16;
    pl.G = (int)spans; pl.short_tiles = kShortTiles;
}

// The same core with workgroups of twice the work or more: what fills a compute unit's LDS (eight tiles at d_m 512, six at 768,
// four at 1024) and, beyond 16 rows, 32 of them, where all of those run at once and the smaller ones would not.  Half the pieces and
// half the expanded queries to receive or less, against a longer way through each workgroup.  Whole steps in bf16, the streaming core
// against this one, a half to the whole of a round (us):
//   d_m 512    8 rows, 32 of 768 to 1024 positions 21.0 / 19.4, 25 of them 20.4 / 17.4    32 rows, 64 of 256 to 512 23.7 / 23.4 (fp16 23.2 / 23.0),
//              25 of 768 to 1024 23.5 / 21.0    40 rows, 30 of 384 to 512 24.2 / 20.9    64 rows, 30 of 300 to 500 25.4 / 22.3
//   d_m 768    12 rows, 60 of 285 to 380 24.0 / 22.4    24 rows, 42 of 427 to 570 27.7 / 26.0    48 rows, 18 of them 25.5 / 22.7    60 rows, 40 of 200 to
//              280 32.0 / 26.7    72 rows, 20 of 285 to 380 28.9 / 25.1
//   d_m 1024   32 rows, 64 of 144 to 192 29.4 / 27.1    64 rows, 31 of 192 to 256 29.8 / 27.6, 15 of 384 to 512 28.7 / 27.4    96 rows, 20 of 192 to
//              256 30.0 / 27.0    128 rows, 15 of them 30.9 / 26.9
// Beyond one round it loses, also where the second is nearly empty (d_m 768, 48 rows, 40 of 200 to 300 27.8 / 31.5; 12 rows, 160 of 211
// 30.6 / 31.1).  Inside it does so where one row block and many spans of an element have nearly every compute unit read positions of
// its own and leave the merge as many pieces: d_m 1024, 32 rows, 20 of 400 to 700 25.0 / 27.4, 42 of 288 to 384 28.5 / 28.9, but 30 of
// them (180 spans) 26.7 / 25.8 and 60 of 192 to 256 (four spans each) 29.7 / 28.9; d_m 768, 12 rows, 20 of 750 to 1000 (eleven) 22.2 / 22.5, 25 of
// 675 to 900 (ten) 23.8 / 23.1.
// A second round of the smaller workgroups (elements of one span) gives way to one of these at d_m 768 (100 of 64, 48 rows, 30.3 / 28.8;
// 128 of 16, 60 rows, 29.8 / 29.6), and at 1024 where 32-row blocks pad no further than 16-row ones (64 rows, 128 of 64 38.1 / 37.1, but 48
// rows 34.3 / 34.8); at 512 two of the smaller ones share a compute unit (200 of 64, 32 rows, 26.1 / 28.2).
// Nor where the streaming core has an element on nearly every compute unit and nothing crosses: single queries over histories, which
// are of one length as a rule, d_m 512, fp16 (bf16): 256 of 128 positions 20.4 / 21.0 (20.9 / 21.3), 256 of 108 20.0 / 20.5 (20.4 /
// 20.8); as graph replays 254 of 128 21.0 / 21.5 (21.5 / 21.8), 248 21.3 / 21.3 (21.5 / 21.8), 236 21.1 / 20.9; 230, where spans cross,
// 22.4 / 20.3 (22.8 / 20.6), and so would 256 of mixed length, 64 to 128, 22.7 / 20.0.  Two and three queries over inputs of one length lose as
// much in fp16 (256 of 128, 16 rows, 23.4 / 23.7, 24 rows 28.4 / 29.1; bf16 24.2 / 23.9, 29.5 / 29.7), but inputs differ in length as a rule,
// and 256 of 64 to 128 gain: 16 rows 25.3 / 23.2, 24 rows 31.0 / 27.8; four gain either way (128 each, 30.5 / 30.0).
static void plan_wide_spans(const Problem &p, int num_cus, int max_slots, CorePlan &pl)
{
    if (p.B > kScanMax) return;
    const int tiles = p.d_m == 512 ? 8 : p.d_m == 768 ? 6 : 4, rg = p.R > 16 ? 2 : 1;
    if (tiles == kShortTiles && rg == 1) return;                         // (nothing wider)
    const int per_element = (p.n + 16 * tiles - 1) / (16 * tiles), blocks = (p.R + 16 * rg - 1) / (16 * rg);
    const long spans = (long)p.B * per_element;
    if (spans > kSpanMax || spans > max_slots || spans * blocks > num_cus || per_element > 13) return;
    if (blocks == 1 && p.d_m == 1024 && per_element > 4 && 4 * spans > 3L * num_cus) return;
    if (rg == 1 && p.d_m == 768 && per_element > 10) return;
    if (p.d_m == 512 && p.beam == 1 && per_element == 1 && 16 * spans > 15L * num_cus) return;
    if (pl.short_tiles) {
        if ((long)pl.G * pl.nblocks <= num_cus || p.d_m == 512) return;
        if (p.d_m == 1024 && 2 * blocks != pl.nblocks) return;
    }
    pl.nrg = pl.block_groups = rg; pl.nblocks = blocks; pl.Rs = blocks * 16 * rg;
    pl.G = (int)spans; pl.short_tiles = tiles;
}

CorePlan plan_core_mfma(const Problem &p, int splits_override, int nrg_override, int num_cus, int max_slots, bool wide)
{
    CorePlan pl = plan_stream(p, splits_override, nrg_override, num_cus, max_slots);
    if (!splits_override && !nrg_override) {
        plan_short_spans(p, num_cus, max_slots, pl);
        if (wide) plan_wide_spans(p, num_cus, max_slots, pl);
    }
    return pl;
}

CutArgs cut_args(const Problem &p, const CorePlan &pl, const Workspace &ws)
{
    CutArgs c;
    c.lengths = p.lengths; c.spans = ws.spans; c.pieces = ws.pieces;
    c.n = p.n; c.B = p.B; c.G = pl.G; c.kcost = pl.kcost; c.short_tiles = pl.short_tiles;
    return c;
}

PieceMap piece_map(const Workspace &ws)
{
    PieceMap m;
    m.table = ws.pieces; m.parts = 1;
    return m;
}

__global__ void __launch_bounds__(64 * kCutWaves) k_cut(const CutArgs c)
{
    __shared__ CutScratch t;
    CutLengths len;
    const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    load_cut_lengths(c, w, l, len);
    build_cut(c, len, t, w, l);
}

hipError_t launch_cut(const CutArgs &c, hipStream_t s)
{
    hipLaunchKernelGGL(k_cut, dim3(1), dim3(64 * kCutWaves), 0, s, c);
    return hipGetLastError();
}

hipError_t launch_elq_f16(const el_attn_ctx *ctx, const Problem &p, const Workspace &ws, const CorePlan &pl,
                          hipStream_t s)
{
    const dim3 grid((p.d_m + 255) / 256, p.R, p.B), block(256);
    uint16_t *planes = (uint16_t *)ws.ELQ;
    if (p.dtype == EL_F16)
        hipLaunchKernelGGL((k_elq_planes<f16_t, false>), grid, block, 0, s, (const float *)ws.Qp, (const f16_t *)ctx->w.Wk,
                           planes, p.beam, p.d_m, p.d_k, p.hd, p.R, pl.Rs);
    else
        hipLaunchKernelGGL((k_elq_planes<bf16_t, true>), grid, block, 0, s, (const float *)ws.Qp, (const bf16_t *)ctx->w.Wk,
                           planes, p.beam, p.d_m, p.d_k, p.hd, p.R, pl.Rs);
    return hipGetLastError();
}

hipError_t launch_core_mfma(const el_attn_ctx *ctx, const Problem &p, const Workspace &ws, const CorePlan &pl,
                            hipStream_t s, hipEvent_t ev0, hipEvent_t ev1)
{
    StreamArgs a;
    a.H = p.H; a.h_stride = p.H_batch_stride; a.lengths = p.lengths;
    a.elq = (const uint16_t *)ws.ELQ;
    a.Xp = (f16_t *)ws.Xp; a.ML = ws.ML; a.spans = ws.spans;
    a.n = p.n; a.B = p.B; a.R = p.R; a.Rs = pl.Rs; a.nblocks = pl.nblocks; a.G = pl.G; a.num_cus = ctx->num_cus;
    a.next_w[0] = ctx->w.WvP; a.next_w[1] = ctx->w.WoP;      // (a segment's a7 belongs to the merge call, usually soon after)
    // H is read once per step; when a batch of it is larger than the 256 MB memory-side cache, keeping its lines
    // out of the caches leaves them to the data that is re-read and raises the streaming rate (measured, core
    // kernel: 1 GB of per-beam histories 216 -> 184 us; 640 MB shared by two row blocks 149 -> 144 us).  Below
    // that it costs: the second row block of a span then misses what the first one fetched (128 MB: 42.7 -> 44.6 us).
    a.stream_hint = (double)p.B * p.n * p.d_m * 2.0 >= 256.0 * 1024 * 1024 ? 1 : 0;
    if (pl.short_tiles) return launch_core_short(a, p.d_m, p.dtype == EL_BF16, pl.short_tiles, pl.nrg, s, ev0, ev1);
    return launch_core_stream(a, p.d_m, p.dtype == EL_BF16, pl.nrg, s, ev0, ev1);
}

hipError_t launch_merge_exp2(const el_attn_ctx *, const Problem &p, const Workspace &ws, const CorePlan &pl,
                             hipStream_t s)
{
    hipLaunchKernelGGL(k_merge_exp2, dim3((p.d_m + 255) / 256, p.R, p.B), dim3(256), 0, s,
                       (const f16_t *)ws.Xp, (const float *)ws.ML, ws.Xn, p.d_m, p.R, pl.Rs, piece_map(ws));
    return hipGetLastError();
}

} // namespace el
