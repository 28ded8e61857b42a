// MFMA kernels for the projection steps of the EL-attention decode step (steps a1, a2, a6, a7 of Algorithm 3's
// attention routine; group 2 of Table 1 -- O(d_m^2) per query, weight-read bound), for d_k = 64:
//
//   a1 + a2  Qp = (q . W^Q + b^Q) * scale, ELQ_i = Qp_i . (W_i^K)^T     k_qelq   (EL-Q as a high + low pair)
//   a6       A_i = X_i . W_i^V, X merged from the pieces                k_vproj
//   a7       out = A . W^O + c_out                                      k_oproj
//
// All three have one shape.  A workgroup of eight wavefronts owns a 64-column block (a head, or 64 output columns)
// and walks over tiles of 16 rows.  Wavefront w contracts an eighth of the contraction dimension: its slice of the
// block's weights stays in registers for all tiles, in fragments packed at prepare time in the order the matrix
// instruction reads them (a load instruction fetches 1 contiguous KB), and the rows' fragments come straight from
// global memory as well, each byte once per workgroup.  Nothing is staged in LDS; everything a tile needs is
// requested before the first product; the eight partial tiles meet in LDS.  Weights are the instruction's A operand:
// a lane ends up with four consecutive columns of one row.  Where 64-column blocks leave compute units idle (few
// rows), the columns are split further and the rows are read once per part, out of L2.
//
// Storage-dtype operands enter the MFMA exactly (a1 runs in the storage type).  From a2 on everything is fp16: bf16
// weights are converted once at prepare time (exact above 2^-14, |error| <= 2^-25 below), and the intermediates Qp, the
// pieces of X and A are rounded to fp16 once each (2^-12 relative; the measured end-to-end error stays several times
// under the 2e-3 bar).  Accumulation is fp32.
#include <type_traits>
#include "mfma.h"
#include "cut.h"

namespace el {

namespace {

// Workgroup -> (64-column block, part of its columns, group of row tiles).  Workgroup ids that differ by a multiple of
// 8 share an XCD and its L2, so each XCD gets one run of the items in block-major order: it then pulls only its own
// blocks' weights from memory, once, instead of every XCD pulling all of them.
struct Place { int block, part, group; };
__device__ __forceinline__ bool place_of(int blocks, int parts, int groups, int id, Place &p)
{
    const int items = blocks * parts * groups, per_xcd = (items + 7) >> 3;
    const int i = (id & 7) * per_xcd + (id >> 3);
    if (i >= items) return false;
    p.block = i / (parts * groups);
    const int j = i - p.block * (parts * groups);
    p.part = j % parts; p.group = j / parts;
    return true;
}
inline dim3 place_grid(int blocks, int parts, int groups) { return dim3(8 * ((blocks * parts * groups + 7) / 8)); }

// Groups the row tiles are dealt to: as many workgroups as there are compute units, all with the same number of tiles
// up to one.
inline int tile_groups(int tiles, int columns_parts, int num_cus)
{
    const int room = num_cus / columns_parts > 0 ? num_cus / columns_parts : 1;
    const int each = (tiles + room - 1) / room;
    return (tiles + each - 1) / each;
}

} // namespace

// ---------------------------------------------------------------------------------------------
// a1 + a2 of one head (Eq. 9's Q_i (W_i^K)^T): Qp = (q . W_i^Q + b_i^Q) * scale of a 16-row tile goes through LDS in
// fp16 and is contracted with the head's rows of W^K at once; NP 32-column fragments of EL-Q per wavefront (all of
// d_m / 256, or one with the columns split over workgroups).  W^K is packed so that a pair of products leaves eight
// consecutive columns in a lane: its high and low halves are 16-byte stores into the core's fragment order.
// Bound: memory latency up to about 64 rows, the bytes of EL-Q (4 per element) beyond.  One launch against the two it
// replaces (a1 on 32 x 32 tiles staged in LDS, a2 with its 8 KB of weights per workgroup), d_m 1024: 4 rows 10.4 ->
// 4.8 us, 256 rows 15.4 -> 10.3 (4.4 of it the stores, 16.8 MB), 512 rows 23.9 -> 14.6, 1280 rows 47.5 -> 24.2.  The split in
// bf16 by the instruction that converts pairs (split16_pair) instead of some twenty operations a value, which a SIMD's two
// wavefronts had no other work to hide under: 4 rows 4.7 -> 4.4, 240 rows of d_m 768 7.6 -> 6.6, 256 rows 10.7 -> 9.5, 512 rows
// 14.4 -> 13.2, 1280 rows 25.0 -> 20.0.
struct QelqArgs {
    const u4 *Wq;          // storage type, [head][k / 32][column / 16 % 4][lane]
    const u4 *Wk;          // fp16, [head][column / 32][half][k / 32 % 2][lane]
    const void *q;         // [M, d_m] storage type
    const void *bq;        // storage type, may be null
    uint16_t *elq;
    f16_t *Qp;             // [M, d_m], or null if nobody reads it
    CutArgs cut;           // the core's cut is built here as well, under this kernel's memory latency: by a workgroup of its own
    int cut_alone;         // (the first, so that it starts at once) where there is room for one, else by the first one
    float scale;
    int M, x, Rs, groups;
};

template <int DM, bool BF, int NP>
__global__ void __launch_bounds__(512)
k_qelq(const QelqArgs a)
{
    constexpr int KS = DM / 256, HEADS = DM / 64, PARTS = DM / 256 / NP, RS = 68;
    __shared__ __attribute__((aligned(16))) float red[8 * 16 * RS];          // [wavefront][row][column, padded]
    __shared__ __attribute__((aligned(16))) f16_t Ql[16 * 72];               // rows 144 bytes apart
    const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r16 = l & 15, q = l >> 4;
    __shared__ CutScratch cut;
    const bool cuts = blockIdx.x == 0;
    CutLengths cut_len;
    if (cuts) load_cut_lengths(a.cut, w, l, cut_len);
    if (a.cut_alone && cuts) {
        build_cut(a.cut, cut_len, cut, w, l);
        return;
    }
    Place pl;
    if (!place_of(HEADS, PARTS, a.groups, blockIdx.x - a.cut_alone, pl)) return;
    const int head = pl.block, tiles = (a.M + 15) >> 4;

    // Everything is requested in the order in which it is waited for, and nothing is looked at before all of it is under way
    // (requests return in order): the lengths, the bias, the rows, W^Q, W^K.  So the cut is built and the products with W^Q are
    // taken while the rest arrives; with the bias behind the weights, converted at once, both waited for all of them.  A workgroup
    // that also cuts, 64 rows, d_m 1024: 7.5 -> 7.0 us, 128 rows 8.2 -> 7.9; others, 60 rows 7.1 -> 6.7, 512 rows 14.8 -> 14.5.
    // the thread that adds up: row srow, columns scol and scol + 1 of the head
    const int srow = threadIdx.x >> 5, scol = 2 * (threadIdx.x & 31);
    unsigned bias_bits = 0;                              // both as they are stored
    if (a.bq) bias_bits = *(const unsigned *)((const uint16_t *)a.bq + head * 64 + scol);
    u4 xq[KS], wq[KS][4], wk[NP][2][2];
    auto load_rows = [&](int tile) {
        const uint16_t *row = (const uint16_t *)a.q + (size_t)min(16 * tile + r16, a.M - 1) * DM + 8 * q;
#pragma unroll
        for (int s = 0; s < KS; ++s) xq[s] = *(const u4 *)(row + 32 * (KS * w + s));
    };
    load_rows(pl.group);
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int t = 0; t < 4; ++t) wq[s][t] = a.Wq[(((size_t)head * (DM / 32) + KS * w + s) * 4 + t) * 64 + l];
    const int pair0 = (pl.part * 8 + w) * NP;
#pragma unroll
    for (int i = 0; i < NP; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int s = 0; s < 2; ++s) wk[i][h][s] = a.Wk[((((size_t)head * (DM / 32) + pair0 + i) * 2 + h) * 2 + s) * 64 + l];
    if (cuts) build_cut(a.cut, cut_len, cut, w, l);
    float bias[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const uint16_t bits = (uint16_t)(bias_bits >> (16 * e));
        bias[e] = BF ? to_f32(bf16_t{bits}) : to_f32(__builtin_bit_cast(f16_t, bits));
    }

    for (int tile = pl.group; tile < tiles; tile += a.groups) {
        f4 acc[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[t] = Mma<BF>::s16(wq[s][t], xq[s], acc[t]);
#pragma unroll
        for (int t = 0; t < 4; ++t) *(f4 *)(red + (w * 16 + r16) * RS + 16 * t + 4 * q) = acc[t];
        if (tile + a.groups < tiles) load_rows(tile + a.groups);
        __syncthreads();
        {
            f2 sum = f2{0.f, 0.f};
#pragma unroll
            for (int s = 0; s < 8; ++s) sum += *(const f2 *)(red + (s * 16 + srow) * RS + scol);
            const h2 v = h2{(_Float16)((sum[0] + bias[0]) * a.scale), (_Float16)((sum[1] + bias[1]) * a.scale)};
            *(h2 *)(Ql + srow * 72 + scol) = v;
            if (a.Qp && pl.part == 0 && 16 * tile + srow < a.M) *(h2 *)(a.Qp + (size_t)(16 * tile + srow) * DM + head * 64 + scol) = v;
        }
        __syncthreads();
        const int m = 16 * tile + r16;
        u4 qf[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) qf[s] = *(const u4 *)(Ql + r16 * 72 + 32 * s + 8 * q);
        uint16_t *dst = a.elq + elq_frag_index(m / a.x, head * a.x + m % a.x, 32 * pair0 + 8 * q, 0, a.Rs, DM);
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            u4 hi, lo;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                f4 e = Mma<false>::s16(wk[i][h][0], qf[0], f4{0.f, 0.f, 0.f, 0.f});
                e = Mma<false>::s16(wk[i][h][1], qf[1], e);
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    unsigned high, low;
                    split16_pair<BF>(e[2 * k], e[2 * k + 1], high, low);
                    hi[2 * h + k] = high; lo[2 * h + k] = low;
                }
            }
            if (m < a.M) {
                *(u4 *)(dst + i * 1024) = hi;
                *(u4 *)(dst + i * 1024 + 512) = lo;
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Merge of the pieces fused with a6 (A_i = X_i . W_i^V, Eq. 5 / Eq. 8), NT 16-column blocks of a head per workgroup.  The
// products are taken of the pieces themselves, which are fp16 values and enter them exactly, and their results are what
// is weighted (log-sum-exp weights, which a lane works out for its own row):
//     A = sum_p (w_p l_p) (Xhat_p . W^V) / sum_p (w_p l_p),  w_p = 2^(m_p - M).
// So a fragment goes from memory into the matrix instruction, and the merge is one multiply-add per result instead of a
// conversion and one per element of X.  Up to four rounds of pieces are in flight (PC); more are folded in with a running maximum.
//
// The instruction takes 16 rows: 16 query rows with one piece each a round, or (row_shift < 4) 8, 4, 2 or 1 of them with 2, 4,
// 8 or 16 of their pieces side by side, added up over the lanes at the end.  Bound: the 64 bytes a clock that a compute unit
// receives.  A round is 32 KB at d_m 1024, the weights of a whole head 128 KB: with 16 rows a workgroup (4 of them
// there, or 16 with their dozens of pieces) one sentence of ten pieces took 32 KB + 10 x 32 KB, 7.9 us, though three
// quarters of the chip were idle; in single rows, 16 pieces a round, 4.6 us.  16 rows in 4 to 7 pieces 7.0 -> 5.0; 32 rows in
// 8 pieces 7.7 -> 5.3; d_m 768, 20 rows in 5 pieces 6.4 -> 5.0; 1280 rows in 448 pieces of 64 rows (16 rows as before) 18.2 -> 16.6.
// Behind that memory latency in a chain of two: the piece table, then statistics and pieces together.
struct VprojArgs {
    const u4 *Wp;          // (W^V) in fragments: [head][k / 32][column / 16 % 4][lane]
    const f16_t *Xp;       // normalised fp16 pieces [slot, Rs, d_m] in fragment order
    const float *ML;       // [slot, Rs, 2]
    f16_t *A;              // [M, d_m] in fragment order
    const int2 *pieces;    // the piece table of the cut
    int M, x, Rs, groups;
    int row_shift;         // a tile is 1 << row_shift rows
    // segment form (fp32): head outputs with b^V and, per head, the log-sum-exp with Eq. 7's key-bias term, instead of A
    const f16_t *Qp;       // [M, d_m], carrying log2(e)/sqrt(d_k)
    const float *bk32, *bv32;
    float *seg_A, *seg_lse;
};

// Sum (or maximum) over the lanes of 16 that hold the same row, (1 << rs) of them apart; every lane gets it.
template <bool MAX>
__device__ __forceinline__ float over_row(float v, int rs)
{
    auto with = [](float x, float y) { return MAX ? fmaxf(x, y) : x + y; };
    v = with(v, dpp<0x128>(v));                          // row_ror:8, :4, :2, :1
    if (rs <= 2) v = with(v, dpp<0x124>(v));
    if (rs <= 1) v = with(v, dpp<0x122>(v));
    if (rs <= 0) v = with(v, dpp<0x121>(v));
    return v;
}

// SEG: the segment form.  What its log-sum-exp needs but Qp and b^K, the merge has in registers, and the head outputs leave as
// the fp32 sums they are, with b^V.  As a
// kernel of its own that read them back, with one thread per head for the statistics, this took 8.8 us at 128 rows.
// LOOP: several row tiles of 16 per workgroup, as a kernel of its own: together with the single tile's code the widest form spills.
template <int DM, int NT, bool SEG, bool LOOP>
__global__ void __launch_bounds__(512)
k_vproj(const VprojArgs a)
{
    constexpr float kLn2 = 0.6931471805599453f;
    constexpr int KS = DM / 256;                         // 32-wide slices of k per wavefront
    constexpr int PC = LOOP && DM == 1024 ? 3 : 4;       // rounds of pieces in flight (with a fourth the widest form spills)
    __shared__ f4 red[2][8 * NT * 64];
    const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r16 = l & 15, q = l >> 4;
    Place pl;
    if (!place_of(DM / 64, 4 / NT, a.groups, blockIdx.x, pl)) return;
    const int head = pl.block, nb = pl.part;
    const int rs = LOOP ? 4 : a.row_shift, at_once = 16 >> rs;      // rows of a tile 1 << rs, pieces of each that the 16 lanes hold side by side
    const int trow = r16 & ((1 << rs) - 1), piece = r16 >> rs;
    const int tiles = (a.M + (1 << rs) - 1) >> rs;
    int j, slot0, np;
    auto look_up = [&](int tile) {
        const int m = min((tile << rs) + trow, a.M - 1), b = m / a.x;
        j = m - b * a.x;
        const int2 e = a.pieces[b];
        slot0 = e.x; np = e.y;
    };
    look_up(pl.group);
    u4 wv[KS][NT];
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int t = 0; t < NT; ++t)
            wv[s][t] = a.Wp[(((size_t)head * (DM / 32) + KS * w + s) * 4 + nb * NT + t) * 64 + l];
    asm volatile("" ::: "memory");                       // (requested here: the compiler sinks them behind the wait for the piece table, 0.5 us)
    int pieces, rounds;
    bool merged;                                         // (uniform)
    size_t row0;
    const f16_t *x0;
    f2 ml[PC];
    u4 xv[PC][KS];
    auto locate = [&]() {                                // of the tile looked up last
        pieces = np;
        row0 = (size_t)slot0 * a.Rs + head * a.x + j;
        x0 = a.Xp + (size_t)slot0 * a.Rs * DM + frag16_index(head * a.x + j, 32 * KS * w + 8 * q, DM);
        const int most = __builtin_amdgcn_readfirstlane((int)max16((float)pieces));          // pieces among the rows
        rounds = (most + at_once - 1) >> (4 - rs);
        merged = most > 1;
    };
    // C rounds from k0 on into registers, the statistics first: the weights are worked out while the rows arrive
    auto load = [&](auto count, int k0) __attribute__((always_inline)) {
        constexpr int C = decltype(count)::value;
        unsigned step[C];
#pragma unroll
        for (int i = 0; i < C; ++i) {
            step[i] = (unsigned)min((k0 + i) * at_once + piece, pieces - 1) * (unsigned)a.Rs;
            ml[i] = *(const f2 *)(a.ML + (row0 + step[i]) * 2);
        }
#pragma unroll
        for (int i = 0; i < C; ++i)
#pragma unroll
            for (int s = 0; s < KS; ++s) xv[i][s] = *(const u4 *)(x0 + (size_t)step[i] * DM + 512 * s);
    };
    // segment form: b^V of the columns that this wavefront adds up, and for the log-sum-exp the row's projected query and b^K; requested
    // ahead of the tile's pieces (several tiles: Qp and b^K where they are used, registers are short there)
    f4 bv = f4{0.f, 0.f, 0.f, 0.f}, bk[4];
    u4 qp[2];
    auto load_seg = [&](int tile) __attribute__((always_inline)) {
        const int m = min((tile << rs) + trow, a.M - 1);
#pragma unroll
        for (int k = 0; k < 2; ++k) qp[k] = *(const u4 *)(a.Qp + (size_t)m * DM + head * 64 + 16 * q + 8 * k);
#pragma unroll
        for (int k = 0; k < 4; ++k) bk[k] = *(const f4 *)(a.bk32 + head * 64 + 16 * q + 4 * k);
    };
    if (SEG && w < NT) bv = *(const f4 *)(a.bv32 + head * 64 + 16 * (nb * NT + w) + 4 * q);
    if (SEG && !LOOP && nb == 0 && w == 7) load_seg(pl.group);
    if (SEG) asm volatile("" ::: "memory");              // (here, and not where they are used)
    f4 acc[NT];
    float m_run, den;
    auto fold = [&](auto count, int k0) __attribute__((always_inline)) {
        constexpr int C = decltype(count)::value;
        float wt[C], m_new = m_run;
#pragma unroll
        for (int i = 0; i < C; ++i) {
            const bool some = (k0 + i) * at_once + piece < pieces && ml[i][1] > 0.f;         // a piece of this row, and not an empty one
            ml[i] = some ? ml[i] : f2{-INFINITY, 0.f};
            m_new = fmaxf(m_new, ml[i][0]);
        }
        if (k0 > 0) {
            const float c = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - m_new);
            den *= c;
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[t][e] = c != 0.f ? acc[t][e] * c : 0.f;
        }
        m_run = m_new;
#pragma unroll
        for (int i = 0; i < C; ++i) {
            wt[i] = ml[i][1] > 0.f ? __builtin_amdgcn_exp2f(ml[i][0] - m_new) * ml[i][1] : 0.f;
            den += wt[i];
            if (C == 1) wt[i] = merged || wt[i] == 0.f ? wt[i] : 1.f;
        }
#pragma unroll
        for (int i = 0; i < C; ++i) {
            f4 part[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) part[t] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int t = 0; t < NT; ++t) part[t] = Mma<false>::s16(wv[s][t], xv[i][s], part[t]);
            // an empty piece's row was never written, and one whose weight underflows may hold fp16 infinities
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[t][e] = fmaf(wt[i] != 0.f ? part[t][e] : 0.f, wt[i], acc[t][e]);
        }
    };
    // Up to PC rounds in straight code, a copy for each number of them: where they are loaded under branches the compiler has the
    // first product wait for the last piece (256 rows in 191 pieces of 64, whole step: 62.2 -> 61.7 us).
    auto rounds_from = [&](int k0, bool loads, bool folds) __attribute__((always_inline)) {
        auto both = [&](auto count) __attribute__((always_inline)) {
            if (loads) load(count, k0);
            if (folds) fold(count, k0);
        };
        const int c = min(rounds - k0, PC);
        if (c == 1) both(std::integral_constant<int, 1>{});
        else if (c == 2) both(std::integral_constant<int, 2>{});
        else if (PC == 3 || c == 3) both(std::integral_constant<int, 3>{});
        else both(std::integral_constant<int, PC>{});
    };
    auto start = [&]() {
        m_run = -INFINITY; den = 0.f;
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};
    };
    int parity = 0;
    auto finish = [&](int tile, bool merged) __attribute__((always_inline)) {
        if (rs < 4) {                                    // the lanes that share a row
            const float m_all = over_row<true>(m_run, rs), c = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - m_all);   // (one piece: 1)
            den = over_row<false>(den * c, rs);
            m_run = m_all;
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[t][e] = over_row<false>(c != 0.f ? acc[t][e] * c : 0.f, rs);
        }
        if (merged) {
            const float inv = den > 0.f ? 1.0f / den : 0.f;
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[t][e] *= inv;
        }
        if (SEG && nb == 0 && w == 7) {                  // (a wavefront that adds nothing up below)
            const int m = min((tile << rs) + trow, a.M - 1);
            if (LOOP) load_seg(tile);
            float c = 0.f;
#pragma unroll
            for (int k = 0; k < 16; ++k) c = fmaf((float)__builtin_bit_cast(h8, qp[k >> 3])[k & 7], bk[k >> 2][k & 3], c);
            c += __shfl_xor(c, 16, 64);
            c += __shfl_xor(c, 32, 64);
            if (q == 0 && piece == 0 && (tile << rs) + trow < a.M)
                a.seg_lse[(size_t)m * (DM / 64) + head] = den > 0.f ? m_run * kLn2 + logf(den) + c * kLn2 : -INFINITY;
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) red[parity][(w * NT + t) * 64 + l] = acc[t];
        __syncthreads();                                 // (the other buffer was last read before the barrier of the tile before)
        if (w < NT) {
            f4 sum = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < 8; ++s) sum += red[parity][(s * NT + w) * 64 + l];
            const int mm = piece == 0 ? (tile << rs) + trow : a.M;
            if (SEG) {
                const int col = head * 64 + 16 * (nb * NT + w) + 4 * q;
                float *o = a.seg_A + (size_t)mm * DM + col;                    // (the caller's: aligned to 4 bytes)
                if (mm < a.M)
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = sum[e] + bv[e];
            } else if (mm < a.M)
                *(h4 *)(a.A + frag16_index(mm, head * 64 + 16 * (nb * NT + w) + 4 * q, DM)) =
                    h4{(_Float16)sum[0], (_Float16)sum[1], (_Float16)sum[2], (_Float16)sum[3]};
        }
        parity ^= 1;
    };
    locate();
    start();
    if (!LOOP) {
        for (int k0 = 0; k0 < rounds; k0 += PC) rounds_from(k0, true, true);
        finish(pl.group, merged);
        return;
    }
    // The first pieces of a tile are requested before the tile before it is added up, into the registers that its products
    // have just left (whole steps, with the two row tiles in flight of a7: 512 histories of 1024, d_m 1024, 210.7 -> 209.5 us;
    // 1000 rows of d_m 768 67.3 -> 66.6).
    rounds_from(0, true, false);
    for (int tile = pl.group; tile < tiles; tile += a.groups) {
        const bool more = tile + a.groups < tiles;
        if (more) look_up(tile + a.groups);              // the next tile's table entries
        start();
        rounds_from(0, false, true);
        for (int k0 = PC; k0 < rounds; k0 += PC) rounds_from(k0, true, true);
        const bool m = merged;
        if (more) { locate(); rounds_from(0, true, false); }
        finish(tile, m);
    }
}

// ---------------------------------------------------------------------------------------------
// a7: out = A . W^O + bias, NT 16-column blocks of a 64-column block per workgroup.  Bound: memory latency, then the
// bytes of weights and rows through L2.  Against 32 x 32 tiles staged in LDS, d_m 1024: 256 rows 6.0 -> 5.1 us, 512
// rows 10.1 -> 7.4, 1280 rows 20.2 -> 12.0.
struct OprojArgs {
    const u4 *Wp;          // (W^O) in fragments: [column / 64][k / 32][column / 16 % 4][lane]
    const f16_t *A;        // [M, d_m] in fragment order
    const float *bias32;
    void *out;
    int M, groups;
};

template <int DM, int NT, typename TO>
__global__ void __launch_bounds__(512)
k_oproj(const OprojArgs a)
{
    constexpr int KS = DM / 256, RS = 16 * NT + 4, TPR = 512 / 16, CPT = 16 * NT / TPR > 0 ? 16 * NT / TPR : 1;   // threads per row, columns per thread
    __shared__ __attribute__((aligned(16))) float red[2][8 * 16 * RS];       // [wavefront][row][column, padded]
    const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r16 = l & 15, q = l >> 4;
    Place pl;
    if (!place_of(DM / 64, 4 / NT, a.groups, blockIdx.x, pl)) return;
    const int tiles = (a.M + 15) >> 4;
    u4 xa[2][KS], wo[KS][NT];                            // rows of two tiles in flight
    auto load_rows = [&](u4 (&x)[KS], int tile) {
        const f16_t *row = a.A + frag16_index(16 * tile + r16, 32 * KS * w + 8 * q, DM);      // (rows past M: padding, their results are dropped)
#pragma unroll
        for (int s = 0; s < KS; ++s) x[s] = *(const u4 *)(row + 512 * s);
    };
    load_rows(xa[0], pl.group);
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int t = 0; t < NT; ++t)
            wo[s][t] = a.Wp[(((size_t)pl.block * (DM / 32) + KS * w + s) * 4 + pl.part * NT + t) * 64 + l];
    if (pl.group + a.groups < tiles) load_rows(xa[1], pl.group + a.groups);
    const int srow = threadIdx.x / TPR, scol = CPT * (threadIdx.x % TPR), col = pl.block * 64 + pl.part * 16 * NT + scol;
    const bool adds = scol < 16 * NT;
    float bias[CPT];
#pragma unroll
    for (int e = 0; e < CPT; ++e) bias[e] = adds && a.bias32 ? a.bias32[col + e] : 0.f;
    auto one_tile = [&](auto buf_tag, int tile) {
        constexpr int BUF = decltype(buf_tag)::value;
        f4 acc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[t] = Mma<false>::s16(wo[s][t], xa[BUF][s], acc[t]);
#pragma unroll
        for (int t = 0; t < NT; ++t) *(f4 *)(red[BUF] + (w * 16 + r16) * RS + 16 * t + 4 * q) = acc[t];
        if (tile + 2 * a.groups < tiles) load_rows(xa[BUF], tile + 2 * a.groups);
        __syncthreads();                                 // (the other buffer was last read before the barrier of the tile before)
        if (adds) {
            float sum[CPT];
#pragma unroll
            for (int e = 0; e < CPT; ++e) sum[e] = 0.f;
#pragma unroll
            for (int s = 0; s < 8; ++s)
#pragma unroll
                for (int e = 0; e < CPT; ++e) sum[e] += red[BUF][(s * 16 + srow) * RS + scol + e];
            const int m = 16 * tile + srow;
            if (m < a.M) {
                TO *o = (TO *)a.out + (size_t)m * DM + col;
#pragma unroll
                for (int e = 0; e < CPT; ++e) from_f32(sum[e] + bias[e], o + e);
            }
        }
    };
    for (int tile = pl.group; tile < tiles; tile += 2 * a.groups) {
        one_tile(std::integral_constant<int, 0>{}, tile);
        if (tile + a.groups < tiles) one_tile(std::integral_constant<int, 1>{}, tile + a.groups);
    }
}

// ---------------------------------------------------------------------------------------------
// Packing at prepare time
// W [K, N] -> fragments [N / 64][k / 32][n / 16 % 4][lane = 16 (k / 8 % 4) + n % 16][k % 8]
template <typename T, typename TO>
__global__ void k_pack_cols(const T *__restrict__ W, TO *__restrict__ P, int K, int N)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (size_t)K * N) return;
    const int e = i & 7, l = (i >> 3) & 63, t = (i >> 9) & 3;
    const int ks = (int)((i >> 11) % (K / 32)), block = (int)((i >> 11) / (K / 32));
    const T v = W[(size_t)(32 * ks + 8 * (l >> 4) + e) * N + block * 64 + 16 * t + (l & 15)];
    if constexpr (std::is_same<T, TO>::value) P[i] = v;
    else P[i] = (TO)to_f32(v);
}

// W^K [d_m, heads * 64] -> fp16 fragments [head][column / 32][half][k / 32][lane][k % 8]; row n of a half's fragment is
// column 8 (n / 4) + 4 half + n % 4 of the 32, so that the results of both halves are eight consecutive columns
template <typename T>
__global__ void k_pack_wk(const T *__restrict__ W, f16_t *__restrict__ P, int d_m, int hd)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (size_t)d_m * hd) return;
    const int e = i & 7, l = (i >> 3) & 63, s = (i >> 9) & 1, h = (i >> 10) & 1;
    const int pair = (int)((i >> 11) % (d_m / 32)), head = (int)((i >> 11) / (d_m / 32)), n = l & 15;
    const int col = 32 * pair + 8 * (n >> 2) + 4 * h + (n & 3);
    P[i] = (f16_t)to_f32(W[(size_t)col * hd + head * 64 + 32 * s + 8 * (l >> 4) + e]);
}

// W^Q in the storage type, the others in fp16
hipError_t launch_pack(int dtype, PackKind kind, const void *W, void *P, int d_m, hipStream_t s)
{
    const dim3 grid((unsigned)(((size_t)d_m * d_m + 255) / 256)), block(256);
    if (kind == kPackWq) hipLaunchKernelGGL((k_pack_cols<uint16_t, uint16_t>), grid, block, 0, s, (const uint16_t *)W, (uint16_t *)P, d_m, d_m);
    else if (kind == kPackWk) {
        if (dtype == EL_BF16) hipLaunchKernelGGL(k_pack_wk<bf16_t>, grid, block, 0, s, (const bf16_t *)W, (f16_t *)P, d_m, d_m);
        else hipLaunchKernelGGL(k_pack_wk<f16_t>, grid, block, 0, s, (const f16_t *)W, (f16_t *)P, d_m, d_m);
    } else {
        if (dtype == EL_BF16) hipLaunchKernelGGL((k_pack_cols<bf16_t, f16_t>), grid, block, 0, s, (const bf16_t *)W, (f16_t *)P, d_m, d_m);
        else hipLaunchKernelGGL((k_pack_cols<f16_t, f16_t>), grid, block, 0, s, (const f16_t *)W, (f16_t *)P, d_m, d_m);
    }
    return hipGetLastError();
}

// Transpose a [rows, cols] matrix of 16- or 32-bit elements.
template <typename E>
__global__ void k_transpose(const E *__restrict__ src, E *__restrict__ dst, int rows, int cols)
{
    __shared__ E tile[32][33];
    const int bx = blockIdx.x * 32, by = blockIdx.y * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 32 x 8
    for (int i = ty; i < 32; i += 8)
        if (by + i < rows && bx + tx < cols) tile[i][tx] = src[(size_t)(by + i) * cols + bx + tx];
    __syncthreads();
    for (int i = ty; i < 32; i += 8)
        if (bx + i < cols && by + tx < rows) dst[(size_t)(bx + i) * rows + by + tx] = tile[tx][i];
}

hipError_t launch_transpose(size_t elem, const void *src, void *dst, int rows, int cols, hipStream_t s)
{
    const dim3 grid((cols + 31) / 32, (rows + 31) / 32), block(256);
    if (elem == 2) hipLaunchKernelGGL(k_transpose<uint16_t>, grid, block, 0, s, (const uint16_t *)src, (uint16_t *)dst, rows, cols);
    else hipLaunchKernelGGL(k_transpose<uint32_t>, grid, block, 0, s, (const uint32_t *)src, (uint32_t *)dst, rows, cols);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
bool gemm_mfma_supported(int dtype, int d_m, int d_k)
{
    return (dtype == EL_F16 || dtype == EL_BF16) && (d_m == 512 || d_m == 768 || d_m == 1024) && d_k == 64;
}

template <int DM, bool BF>
static void launch_qelq_t(QelqArgs &a, int num_cus, hipStream_t s)
{
    constexpr int FULL = DM / 256;
    const int tiles = (a.M + 15) / 16, heads = DM / 64;
    // the columns of EL-Q split over FULL workgroups while all of them run at once
    const int parts = tiles * heads * FULL <= num_cus ? FULL : FULL == 4 && tiles * heads * 2 <= num_cus ? 2 : 1;
    a.groups = tile_groups(tiles, heads * parts, num_cus);
    dim3 grid = place_grid(heads, parts, a.groups), block(512);
    a.cut_alone = (int)grid.x < num_cus || DM == 512 ? 1 : 0;
    grid.x += a.cut_alone;     // (d_m 512: two workgroups fit a compute unit's registers)
    if (parts == 1) hipLaunchKernelGGL((k_qelq<DM, BF, FULL>), grid, block, 0, s, a);
    else if (FULL == 4 && parts == 2) hipLaunchKernelGGL((k_qelq<DM, BF, FULL == 4 ? 2 : 1>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_qelq<DM, BF, 1>), grid, block, 0, s, a);
}

// a1 + a2: ELQ[b, i*beam+j, :] = ((q . W_i^Q + b_i^Q) * scale) . (W_i^K)^T      high + low planes in fragment order, pl.Rs
// rows per b; Qp [B*beam, hd] fp16 as well if `keep_qp`
hipError_t launch_qelq_mfma(const el_attn_ctx *ctx, const Problem &p, const Workspace &ws, const CorePlan &pl, float scale, bool keep_qp, hipStream_t s)
{
    QelqArgs a;
    a.cut = cut_args(p, pl, ws);
    a.Wq = (const u4 *)ctx->w.WqP; a.Wk = (const u4 *)ctx->w.WkP; a.q = p.queries; a.bq = ctx->w.bq;
    a.elq = (uint16_t *)ws.ELQ; a.Qp = keep_qp ? (f16_t *)ws.Qp : nullptr; a.scale = scale;
    a.M = p.B * p.beam; a.x = p.beam; a.Rs = pl.Rs;
    const bool bf = p.dtype == EL_BF16;
    if (p.d_m == 1024) { if (bf) launch_qelq_t<1024, true>(a, ctx->num_cus, s); else launch_qelq_t<1024, false>(a, ctx->num_cus, s); }
    else if (p.d_m == 768) { if (bf) launch_qelq_t<768, true>(a, ctx->num_cus, s); else launch_qelq_t<768, false>(a, ctx->num_cus, s); }
    else { if (bf) launch_qelq_t<512, true>(a, ctx->num_cus, s); else launch_qelq_t<512, false>(a, ctx->num_cus, s); }
    return hipGetLastError();
}

// merge + a6: A[b*beam+j, head i] = (sum_p w_p Xp[b,p,i*beam+j,:]) . W_i^V       fp16
template <int DM, bool SEG>
static void launch_vproj_t(VprojArgs &a, int pieces, int num_cus, hipStream_t s)
{
    const int heads = DM / 64;
    // Rows and columns of a workgroup: whatever makes a compute unit receive least, in units of a round of pieces (a whole
    // head's weights are four), while all workgroups run at once; 16 rows and the fewest column parts beyond that.  One sentence
    // of 613 positions (10 pieces, 4 rows, d_m 1024): 16 rows 7.0 us, 4 rows 4.9, 1 row 4.6; one piece: 16 rows 3.7 us, 1 row 3.9.
    auto tiles_of = [&](int rs) { return (a.M + (1 << rs) - 1) >> rs; };
    int parts = 1, shift = 4, least = 0;
    for (int rs = 4; rs >= 0; --rs)
        for (int p = 4; p >= 1; p >>= 1) {
            const int at_once = 16 >> rs;
            if ((p > 1 || rs < 4) && tiles_of(rs) * heads * p > num_cus) continue;
            const int cost = 4 / p + (pieces + at_once - 1) / at_once;
            if (least == 0 || cost < least) { least = cost; parts = p; shift = rs; }
        }
    a.row_shift = shift;
    a.groups = tile_groups(tiles_of(shift), heads * parts, num_cus);
    const dim3 grid = place_grid(heads, parts, a.groups), block(512);
    if (parts == 4) hipLaunchKernelGGL((k_vproj<DM, 1, SEG, false>), grid, block, 0, s, a);
    else if (parts == 2) hipLaunchKernelGGL((k_vproj<DM, 2, SEG, false>), grid, block, 0, s, a);
    else if (tiles_of(shift) <= a.groups) hipLaunchKernelGGL((k_vproj<DM, 4, SEG, false>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_vproj<DM, 4, SEG, true>), grid, block, 0, s, a);
}

hipError_t launch_vproj_mfma(const el_attn_ctx *ctx, const Problem &p, const Workspace &ws, const CorePlan &pl,
                             const SegOut *seg, hipStream_t s)
{
    VprojArgs a;
    a.Wp = (const u4 *)ctx->w.WvP; a.Xp = (const f16_t *)ws.Xp; a.ML = ws.ML; a.A = (f16_t *)ws.A;
    a.pieces = ws.pieces;
    a.M = p.B * p.beam; a.x = p.beam; a.Rs = pl.Rs;
    a.Qp = (const f16_t *)ws.Qp; a.bk32 = ctx->w.bk32; a.bv32 = ctx->w.bv32;
    a.seg_A = seg ? seg->A : nullptr; a.seg_lse = seg ? seg->lse : nullptr;
    // pieces of the longest element, about
    const int pieces = pl.short_tiles ? pl.G / p.B : pl.G > p.B ? (pl.G + p.B - 1) / p.B + 1 : 1;
    if (p.d_m == 1024) { if (seg) launch_vproj_t<1024, true>(a, pieces, ctx->num_cus, s); else launch_vproj_t<1024, false>(a, pieces, ctx->num_cus, s); }
    else if (p.d_m == 768) { if (seg) launch_vproj_t<768, true>(a, pieces, ctx->num_cus, s); else launch_vproj_t<768, false>(a, pieces, ctx->num_cus, s); }
    else { if (seg) launch_vproj_t<512, true>(a, pieces, ctx->num_cus, s); else launch_vproj_t<512, false>(a, pieces, ctx->num_cus, s); }
    return hipGetLastError();
}

// a7: out = A . W^O + bias
template <int DM, typename TO>
static void launch_oproj_t(OprojArgs &a, int num_cus, hipStream_t s)
{
    const int tiles = (a.M + 15) / 16, blocks = DM / 64;
    const int parts = tiles * blocks * 4 <= num_cus ? 4 : tiles * blocks * 2 <= num_cus ? 2 : 1;
    a.groups = tile_groups(tiles, blocks * parts, num_cus);
    const dim3 grid = place_grid(blocks, parts, a.groups), block(512);
    if (parts == 4) hipLaunchKernelGGL((k_oproj<DM, 1, TO>), grid, block, 0, s, a);
    else if (parts == 2) hipLaunchKernelGGL((k_oproj<DM, 2, TO>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_oproj<DM, 4, TO>), grid, block, 0, s, a);
}

template <typename TO>
static void launch_oproj_d(OprojArgs &a, int d_m, int num_cus, hipStream_t s)
{
    if (d_m == 1024) launch_oproj_t<1024, TO>(a, num_cus, s);
    else if (d_m == 768) launch_oproj_t<768, TO>(a, num_cus, s);
    else launch_oproj_t<512, TO>(a, num_cus, s);
}

hipError_t launch_oproj_mfma(const el_attn_ctx *ctx, const Problem &p, const Workspace &ws, const float *bias32, hipStream_t s)
{
    OprojArgs a;
    a.Wp = (const u4 *)ctx->w.WoP; a.A = (const f16_t *)ws.A; a.bias32 = bias32; a.out = p.out;
    a.M = p.B * p.beam;
    if (p.out_dtype == EL_F32) launch_oproj_d<float>(a, p.d_m, ctx->num_cus, s);
    else if (p.out_dtype == EL_BF16) launch_oproj_d<bf16_t>(a, p.d_m, ctx->num_cus, s);
    else launch_oproj_d<f16_t>(a, p.d_m, ctx->num_cus, s);
    return hipGetLastError();
}

} // namespace el
