// MFMA attention core for short spans, steps a3-a5 of the EL-attention decode step (Eq. 9 with K = V = H), gfx950.
//
// A workgroup takes at most NTM 16-row tiles of one batch element (cut.h deals every element out to such spans) and 16 RG
// expanded-query rows: four tiles and 16 rows, or, where that is more workgroups than the chip holds, as many tiles as LDS holds and
// up to 32 rows (plan_wide_spans).  It has no loop over tiles: the whole span is requested at once, straight into LDS, its scores are
// taken, one softmax, the weighted sum, and the piece leaves.  Where the streaming core (core_stream.hip) would have a few
// tiles per workgroup, most of its time is the latency of its pipeline: a step per tile and two more, each as long as the
// chain from one exchange to the next, 0.8 us, whatever the tile holds.
//
// Eight wavefronts; each owns an eighth of the model dimension, for the scores as for the weighted sum, so the tiles stay in
// the wavefront that fetched them (no barrier waits for another one's fetches) and only scores and probabilities meet:
//   scores        S^T[t, r] partial over the slice, 16x16x32 MFMA in the storage type, A = H rows, B = EL-Q as a high + low pair
//   softmax       a wavefront per four rows sums the eight partials of the positions: fp32, one maximum, one sum
//   weighted sum  X^T[d, r] over the slice's columns, 16x16x32 MFMA (two tiles deep), A = H columns through the transposing LDS
//                 read, B = P (fp16, or a high + low bf16 pair).  The column fragments are read together with the scores'
//                 operands, so that the tiles' part of LDS is free for the partial scores.
// Kernel times, streaming core -> here, d_m 1024: one sentence of 613 positions, 64 rows (40 workgroups) 10.2 -> 6.3 us; 4 of 205
// to 410 10.0 -> 6.6; 8 of 512 (256 workgroups) 13.9 -> 9.5; 128 histories of 37, 16 rows, 9.7 -> 6.4.  More pieces take some of it
// back in the merge (one sentence: ten instead of eight, 4.0 -> 4.6).
// The tiles' fragments are read while EL-Q arrives and all partial scores of a position before any is added, instead of everything behind
// one wait and the partials two by two: whole steps of 96 shapes of one to eight spans an element 1.014 times as fast (0.99 to
// 1.04), one sentence of 613 positions 17.06 -> 16.62 us, twelve layers 243.7 -> 238.3.
// Bound: memory latency (the table of the cut, then tiles and EL-Q together), then the 64 bytes a clock that a compute unit
// receives: at d_m 1024 128 KB of tiles and 64 KB of EL-Q (128 KB with 32 rows).  Behind the wait a wavefront of a wide workgroup of 32
// rows has 64 products for the scores instead of 16 at d_m 512, 72 instead of 24 at 768 and 64 instead of 32 at 1024, in groups of four
// tiles (two at 1024), so that their results and operands fit the registers.
#include <type_traits>
#include <hip/hip_ext.h>
#include "mfma.h"

namespace el {

namespace {

constexpr int kWaves = 8;

// A wavefront's slice of a tile lies in LDS as windows of 64 columns (16 rows of 128 bytes), and one of 32 (16 rows of 64
// bytes) where the slice is 96 columns.  Chunk (16 bytes) c of row r is at chunk position c ^ swizzle(r): 16 rows of one chunk
// (a score operand) and eight rows of two (half a wavefront's transposing read) hit every bank once.
__device__ __forceinline__ int swizzle64(int row) { return (((row >> 1) & 1) << 2) | ((row >> 2) & 3); }
__device__ __forceinline__ int swizzle32(int row) { return (row >> 2) & 3; }

} // namespace

template <int DM, bool BF16, int NTM, int RG>
__global__ void __launch_bounds__(64 * kWaves)
k_core_short(const StreamArgs a)
{
    constexpr int kPos = kTile * NTM;               // positions of a span
    constexpr int ROWB = DM * 2;                    // bytes per row of H
    constexpr int CW = DM / kWaves;                 // columns of a wavefront: 128, 96 or 64
    constexpr int CHK = CW / 32;                    // 32-column chunks of them
    constexpr int WIN = CW / 64;                    // windows of 64 columns
    constexpr bool HALF = CW % 64 != 0;             // and one of 32 (d_m 768)
    constexpr int MB = CW / 16;                     // 16-column blocks of the weighted sum
    constexpr int WSL = CW * 2 * kTile;             // bytes of a wavefront's slice of a tile
    constexpr int NI = WSL / 1024;                  // fetch instructions per wavefront and tile
    constexpr int NP = BF16 ? 2 : 1;                // 16-bit planes of P
    constexpr int ROWS = 16 * RG;
    constexpr bool PAD = NTM == 6;                  // rows of 96 positions do not swizzle: 16 bytes of padding instead
    constexpr int SRS = kPos * 4 + (PAD ? 16 : 0), PRS = kPos * 2 + (PAD ? 16 : 0);     // row strides of partial scores and of P
    static_assert((NTM == 4 || NTM == 6 || NTM == 8) && ROWS * SRS <= NTM * WSL, "the partial scores take the place of the tiles");

    __shared__ __attribute__((aligned(1024))) char T[kWaves * NTM * WSL];  // [wavefront][tile][window]; then partial scores [wavefront][row][position]
    __shared__ __attribute__((aligned(16))) char Px[NP * ROWS * PRS];         // probabilities [plane][row][position]
    __shared__ float Linv[ROWS];

    const int tid = threadIdx.x, l = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = l & 15, g = l >> 4;

    // workgroup -> (span, row block), as in the streaming core: what shares tiles or expanded queries shares an XCD
    const int nwg = a.G * a.nblocks, per_xcd = (nwg + 7) >> 3;
    if (blockIdx.x >= 8 * per_xcd) { read_ahead<DM>(a, per_xcd); return; }
    const int place = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (place >= nwg) return;
    const int span = place / a.nblocks, row0 = (place - span * a.nblocks) * ROWS;
    typedef int i8v __attribute__((ext_vector_type(8)));
    const i8v sp = ((const __attribute__((address_space(4))) i8v *)(uintptr_t)a.spans)[span];     // (a scalar load: the table was written by an earlier kernel)
    const int b = sp[0], nt = sp[2], slot = sp[3];
    if (nt <= 0) return;                            // an element with fewer tiles than the longest one has fewer spans
    const int valid = min(sp[4] - sp[1] * kTile, nt * kTile);          // positions of the span that exist

    // ---- requests: 1 KB per instruction, lane l landing at chunk position l.  A window of 64 columns is two of 8 rows x 128 bytes,
    // the one of 32 columns one of 16 rows x 64 bytes.  A row that does not exist is replaced by the last valid one (never by
    // memory past the length): its scores are masked and its probabilities exactly zero.
    const EL_LDS(char) *Tw = (const EL_LDS(char) *)T + w * (NTM * WSL);
    const unsigned t_lds = (unsigned)(uintptr_t)Tw;
    const char *src = (const char *)a.H + (HALF ? w * 128 : w * CW * 2) + ((size_t)b * a.h_stride * 2 + (size_t)sp[1] * kTile * ROWB);
#pragma unroll
    for (int t = 0; t < NTM; ++t) {
        if (t >= nt) continue;                      // (uniform)
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            unsigned off;
            if (HALF && j == 2 * WIN) {
                const int r = l >> 2;
                off = (unsigned)(min(kTile * t + r, valid - 1) * ROWB + (((l & 3) ^ swizzle32(r)) << 4) + 1024 - 64 * w);
            } else {
                const int r = (l >> 3) + 8 * (j & 1);
                off = (unsigned)(min(kTile * t + r, valid - 1) * ROWB + (((l & 7) ^ swizzle64(r)) << 4) + 128 * (j >> 1));
            }
            dma_piece(t_lds + t * WSL + 1024 * j, off, src);
        }
    }
    // this wavefront's slice of EL-Q (fragment order, low plane 1 KB after the high one).  Rows beyond R are whatever the workspace
    // holds: they only reach their own row's scores, which nobody reads.
    auto chunk32 = [&](int c) __attribute__((always_inline)) { return HALF && c == 2 * WIN ? 16 + w : HALF ? 2 * w + c : CHK * w + c; };   // which 32 columns of d_m
    u4 elq[CHK][RG][2];
    {
        const char *e = (const char *)a.elq + elq_frag_index(b, row0 + r16, 8 * g, 0, a.Rs, DM) * 2;
#pragma unroll
        for (int c = 0; c < CHK; ++c)
#pragma unroll
            for (int rg = 0; rg < RG; ++rg)
#pragma unroll
                for (int pl = 0; pl < 2; ++pl) elq[c][rg][pl] = *(const u4 *)(e + rg * (DM / 32) * 2048 + chunk32(c) * 2048 + pl * 1024);
    }
    // The tiles have landed when only the EL-Q loads, requested last, are under way (requests return in order): the fragments of scores
    // and weighted sum are read while those arrive, and the products of a chunk of columns wait for its own two planes alone.
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(2 * CHK * RG) : "memory");

    // ---- scores, and the column fragments of the weighted sum ----
    const int s_addr = r16 * 128 + ((g ^ swizzle64(r16)) << 4);                        // chunk c of window c / 2; odd c: ^ 64
    const int s_addr2 = 2048 * WIN + r16 * 64 + ((g ^ swizzle32(r16)) << 4);
    // Fragment of columns 16 mb .. of two tiles: lane 16 g + i (i = 4 k + q) reads rows 8 (g & 1) + k (and + 4) of tile 2 u + g / 2,
    // columns 4 q .. + 3.
    s4 tb[NTM / 2][MB][2];
    const int tr = 8 * (g & 1) + (r16 >> 2), tq = r16 & 3;
    const int x64 = tr * 128 + (((tq >> 1) ^ swizzle64(tr)) << 4) + (tq & 1) * 8;              // block mb of a window: ^ 32 (mb & 3); row + 4: + 512, ^ 16
    const int x32 = 2048 * WIN + tr * 64 + (((tq >> 1) ^ swizzle32(tr)) << 4) + (tq & 1) * 8;  // ^ 32 (mb & 1); row + 4: + 256, ^ 16
    // In straight code for all tiles or for fewer: a tile that does not exist is replaced by the last one (behind branches a product
    // waits for more reads than its own).
    auto scores = [&](auto count) __attribute__((always_inline)) {
        constexpr int NTL = decltype(count)::value, GRP = DM == 1024 && RG == 2 ? 2 : 4;      // tiles whose products run side by side
        f4 sum[NTL][RG];
#pragma unroll
        for (int t0 = 0; t0 < NTL; t0 += GRP) {
            constexpr int N = NTL < GRP ? NTL : GRP;
            u4 hb[N][CHK];
#pragma unroll
            for (int c = 0; c < CHK; ++c)
#pragma unroll
                for (int t = 0; t < N; ++t) {
                    if (t0 + t >= NTL) continue;
                    const EL_LDS(char) *F = Tw + min(t0 + t, nt - 1) * WSL;
                    hb[t][c] = c < 2 * WIN ? *(const EL_LDS(u4) *)(F + (s_addr ^ (64 * (c & 1))) + 2048 * (c >> 1)) : *(const EL_LDS(u4) *)(F + s_addr2);
                }
#pragma unroll
            for (int u = t0 / 2; u < (t0 + N) / 2; ++u) {
                if (2 * u >= NTL) continue;
                const EL_LDS(char) *F = Tw + min(2 * u + (g >> 1), nt - 1) * WSL;
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) {
                    const int lo = mb < 4 * WIN ? (x64 ^ (32 * (mb & 3))) : (x32 ^ (32 * (mb & 1)));
                    const int at = mb < 4 * WIN ? 2048 * (mb >> 2) : 0;
                    tb[u][mb][0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((EL_LDS(s4) *)(F + lo + at));
                    tb[u][mb][1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((EL_LDS(s4) *)(F + (lo ^ 16) + at + (mb < 4 * WIN ? 512 : 256)));
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            f4 sc[N][RG][2];
#pragma unroll
            for (int t = 0; t < N; ++t)
#pragma unroll
                for (int rg = 0; rg < RG; ++rg) sc[t][rg][0] = sc[t][rg][1] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < CHK; ++c)
#pragma unroll
                for (int rg = 0; rg < RG; ++rg)
#pragma unroll
                    for (int pl = 0; pl < 2; ++pl)
#pragma unroll
                        for (int t = 0; t < N; ++t)
                            if (t0 + t < NTL) sc[t][rg][pl] = Mma<BF16>::s16(hb[t][c], elq[c][rg][pl], sc[t][rg][pl]);
#pragma unroll
            for (int t = 0; t < N; ++t)
#pragma unroll
                for (int rg = 0; rg < RG; ++rg)
                    if (t0 + t < NTL) sum[t0 + t][rg] = sc[t][rg][0] + sc[t][rg][1];
        }
        // exchange: partial scores where this wavefront's tiles were (read by now); chunk (four positions) c of row r at c ^ r % 16
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int t = 0; t < NTL; ++t)
#pragma unroll
            for (int rg = 0; rg < RG; ++rg)
                *(f4 *)(T + w * (NTM * WSL) + (16 * rg + r16) * SRS + ((PAD ? 4 * t + g : (4 * t + g) ^ r16) << 4)) = sum[t][rg];
    };
    constexpr int FEW = NTM == 4 ? 2 : 4;
    if (nt > FEW) scores(std::integral_constant<int, NTM>{});
    else scores(std::integral_constant<int, FEW>{});
    __syncthreads();
    // ---- softmax: four rows per wavefront, a lane's positions in chunks of four, 64 apart ----
    if (w < ROWS / 4) {
        constexpr int NC = kPos / 4, CL = (NC + 15) / 16;                // chunks of a row, and of a lane
        const int srow = 4 * w + g;
        f4 s[CL], part[kWaves][CL];
        auto chunk = [&](int j) { return NC % 16 != 0 && j == CL - 1 ? min(r16 + 16 * j, NC - 1) : r16 + 16 * j; };   // (a lane without a last chunk: some chunk)
        auto here = [&](int j) { return NC % 16 == 0 || j < CL - 1 || r16 + 16 * j < NC; };
#pragma unroll
        for (int j = 0; j < CL; ++j)
#pragma unroll
            for (int p = 0; p < kWaves; ++p) part[p][j] = *(const f4 *)(T + p * (NTM * WSL) + srow * SRS + ((PAD ? chunk(j) : chunk(j) ^ (srow & 15)) << 4));
        __builtin_amdgcn_sched_barrier(0);           // (left to itself the compiler reads two at a time and waits for them)
        float mx = kMasked;
#pragma unroll
        for (int j = 0; j < CL; ++j) {
            s[j] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int p = 0; p < kWaves; ++p) s[j] += part[p][j];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                s[j][e] = 4 * (r16 + 16 * j) + e < valid ? s[j][e] : kMasked;               // positions at or beyond the length do not exist
                mx = fmaxf(mx, s[j][e]);
            }
        }
        mx = max16(mx);
        float sum = 0.f;
#pragma unroll
        for (int j = 0; j < CL; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) { s[j][e] = __builtin_amdgcn_exp2f(s[j][e] - mx); sum += s[j][e]; }
        sum = sum16(sum);
#pragma unroll
        for (int j = 0; j < CL; ++j) {
            if (!here(j)) continue;
            // 16-byte chunk c of a row of P at c ^ (row / 2) % 8
            const int c = r16 + 16 * j;
            char *dst = Px + srow * PRS + ((PAD ? c >> 1 : (c >> 1) ^ ((srow >> 1) & 7)) << 4) + (c & 1) * 8;
            if (BF16) {
                // p = high + low, both bf16 by truncation
                unsigned hi[4], lo[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    hi[e] = __float_as_uint(s[j][e]) & 0xffff0000u;
                    lo[e] = __float_as_uint(s[j][e] - __uint_as_float(hi[e]));
                }
                *(u2 *)dst = u2{(hi[0] >> 16) | hi[1], (hi[2] >> 16) | hi[3]};
                *(u2 *)(dst + (NP - 1) * ROWS * PRS) = u2{(lo[0] >> 16) | (lo[1] & 0xffff0000u), (lo[2] >> 16) | (lo[3] & 0xffff0000u)};
            } else
                *(u2 *)dst = u2{__builtin_bit_cast(unsigned, __builtin_convertvector(f2{s[j][0], s[j][1]}, h2)), __builtin_bit_cast(unsigned, __builtin_convertvector(f2{s[j][2], s[j][3]}, h2))};
        }
        if (r16 == 0) {
            Linv[srow] = sum > 0.f ? 1.0f / sum : 0.f;
            if (row0 + srow < a.R) {
                float *ml = a.ML + ((size_t)slot * a.Rs + row0 + srow) * 2;
                ml[0] = mx; ml[1] = sum;
            }
        }
    }
    __syncthreads();
    // ---- weighted sum ----
    f4 X[RG][MB];
#pragma unroll
    for (int rg = 0; rg < RG; ++rg)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) X[rg][mb] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < NTM / 2; ++u) {
        if (2 * u >= nt) continue;
        u4 P[RG][NP];
#pragma unroll
        for (int rg = 0; rg < RG; ++rg)
#pragma unroll
            for (int pl = 0; pl < NP; ++pl)
                P[rg][pl] = *(const u4 *)(Px + (pl * ROWS + 16 * rg + r16) * PRS + ((PAD ? 4 * u + g : (4 * u + g) ^ (r16 >> 1)) << 4));
#pragma unroll
        for (int rg = 0; rg < RG; ++rg)
#pragma unroll
            for (int pl = 0; pl < NP; ++pl)
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) {
                    const s4 lo = tb[u][mb][0], hi = tb[u][mb][1];
                    X[rg][mb] = Mma<BF16>::s16(__builtin_bit_cast(u4, s8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]}), P[rg][pl], X[rg][mb]);
                }
    }
    // ---- the piece: normalised, fp16, in fragment order.  A lane holds columns 4 g .. + 3 of every 16-column block of its row; the
    // lanes of neighbouring groups trade (v_permlane16_swap), so that each stores eight consecutive columns of one block.
#pragma unroll
    for (int rg = 0; rg < RG; ++rg) {
        const int row = row0 + 16 * rg + r16;
        const float inv = Linv[16 * rg + r16];
        f16_t *x_out = a.Xp + (size_t)slot * a.Rs * DM + frag16_index(row, 16 * (g & 1) + 8 * (g >> 1), DM);
#pragma unroll
        for (int c = 0; c < CHK; ++c) {
            unsigned lo[2], hi[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                lo[h] = __builtin_bit_cast(unsigned, __builtin_convertvector(f2{X[rg][2 * c][2 * h] * inv, X[rg][2 * c][2 * h + 1] * inv}, h2));
                hi[h] = __builtin_bit_cast(unsigned, __builtin_convertvector(f2{X[rg][2 * c + 1][2 * h] * inv, X[rg][2 * c + 1][2 * h + 1] * inv}, h2));
                const auto sw = __builtin_amdgcn_permlane16_swap(lo[h], hi[h], false, false);
                lo[h] = sw[0]; hi[h] = sw[1];
            }
            if (row < a.R) *(u4 *)(x_out + 512 * chunk32(c)) = u4{lo[0], lo[1], hi[0], hi[1]};
        }
    }
}

// (a pair of events is carried by the launch itself)
template <int DM, bool BF16, int NTM, int RG>
static hipError_t launch_t(const StreamArgs &a, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1)
{
    const dim3 grid = core_grid(a);
    if (ev0 && ev1) hipExtLaunchKernelGGL((k_core_short<DM, BF16, NTM, RG>), grid, dim3(512), 0, s, ev0, ev1, 0, a);
    else hipLaunchKernelGGL((k_core_short<DM, BF16, NTM, RG>), grid, dim3(512), 0, s, a);
    return hipGetLastError();
}

template <int DM, bool BF16, int WIDE>
static hipError_t launch_d(const StreamArgs &a, int tiles, int rg, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1)
{
    if (tiles == kShortTiles && rg == 1) return launch_t<DM, BF16, kShortTiles, 1>(a, s, ev0, ev1);
    if (tiles == WIDE && rg == 2) return launch_t<DM, BF16, WIDE, 2>(a, s, ev0, ev1);
    if constexpr (WIDE > kShortTiles)
        if (tiles == WIDE && rg == 1) return launch_t<DM, BF16, WIDE, 1>(a, s, ev0, ev1);
    return hipErrorInvalidValue;
}

hipError_t launch_core_short(const StreamArgs &a, int d_m, bool bf16, int tiles, int rg, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1)
{
    if (d_m == 1024) return bf16 ? launch_d<1024, true, 4>(a, tiles, rg, s, ev0, ev1) : launch_d<1024, false, 4>(a, tiles, rg, s, ev0, ev1);
    if (d_m == 768) return bf16 ? launch_d<768, true, 6>(a, tiles, rg, s, ev0, ev1) : launch_d<768, false, 6>(a, tiles, rg, s, ev0, ev1);
    if (d_m == 512) return bf16 ? launch_d<512, true, 8>(a, tiles, rg, s, ev0, ev1) : launch_d<512, false, 8>(a, tiles, rg, s, ev0, ev1);
    return hipErrorInvalidValue;
}

} // namespace el
