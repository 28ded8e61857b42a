// How the attention core's work is cut, worked out on the device from the actual lengths by ONE workgroup of eight
// wavefronts: a table of spans (what each workgroup of the core walks) and a table of pieces (where the partial results of a
// batch element are), both read with one load.  The workgroup is one of the launch that precedes the core (k_qelq), which
// does this under its memory latency: in the core, every workgroup repeated the scan of all lengths (1.7 us of every launch
// at 64 batch elements) before it could request its first tile.  A wavefront takes 64 elements (and 64 spans) at a time; as
// the work of one wavefront the cut outlasted that latency where no compute unit is left for it alone: k_qelq, d_m 1024, 512
// rows of as many elements, one wavefront 18.2 us, eight 14.8, and 14.5 since they wait for the lengths alone; the whole step
// with histories of 1024 210.7 -> 207.2 -> 206.6.
#pragma once
#include "el_internal.h"

namespace el {

constexpr int kCutWaves = 8;
constexpr int kCutChunks = kScanMax / 64, kCutMine = kCutChunks / kCutWaves;

// LDS: prefix of tiles, lengths, per span its first tile and its element, and per chunk of 64 elements its tiles and, for two
// guesses, its spans
struct CutScratch { int E[kScanMax + 1], len[kScanMax + 3], first[kSpanMax + 1], owner[kSpanMax], tiles[kCutChunks], count[2][kCutChunks]; };
struct CutLengths { int v[kCutMine]; };              // lane l of wavefront w: lengths of elements 64 (w + 8 c) + l, as the caller wrote them

__device__ __forceinline__ int cut_length(const CutArgs &a, int v) { return min(max(v, 1), a.n); }

// All lengths requested at once, and ahead of whatever else the workgroup has to fetch: by an index that stays inside the
// batch, not in a branch, and looked at in build_cut only.  Clamped and masked here, each was waited for before the next
// request went out, by every wavefront of the one workgroup that the launch waits for.
__device__ __forceinline__ void load_cut_lengths(const CutArgs &a, int w, int l, CutLengths &t)
{
#pragma unroll
    for (int c = 0; c < kCutMine; ++c) t.v[c] = a.n;
    if (a.lengths && a.B <= kScanMax)
#pragma unroll
        for (int c = 0; c < kCutMine; ++c) t.v[c] = a.lengths[min(64 * (w + kCutWaves * c) + l, a.B - 1)];
}

// inclusive scan over the 64 lanes on the vector ALU (row shifts, then the row totals broadcast); no LDS round trips
__device__ __forceinline__ int wave_scan(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);      // lane - 1 of the same 16
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);      // - 2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);      // - 4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);      // - 8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);     // last lane of rows 0 and 2 to rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);     // lane 31 to rows 2 and 3
    return v;
}

// x / y for 0 <= x, 0 < y and a quotient below 2^20 (ry = 1.0f / y): a fraction of the instructions of an integer division
__device__ __forceinline__ int small_quotient(int x, int y, float ry)
{
    int q = (int)((float)x * ry);
    const int r = x - q * y;
    return q + (r >= y ? 1 : 0) - (r < 0 ? 1 : 0);
}

// Executed by a whole workgroup (lane l of wavefront w; it has barriers).  Two ways to cut, the one with the shorter longest span wins:
//   flattened   the 16-row tiles of all elements lie on one axis, element after element, each element preceded by a
//               gap of `kcost` units (what moving on to a new element costs a workgroup, in tiles): tile kt of element
//               b sits at E[b] + kcost (b + 1) + kt.  The axis is cut into G equal spans; span g's piece of element b
//               is slot g + b (unique: along the axis, span and element never decrease and one of them grows).
//   per element every element is cut into its own spans of at most s tiles: nothing crosses, a piece is a span and has
//               its number.  The better one for few elements (one sentence: the flattened axis would start with a gap
//               for nothing), and the only one for the core of short spans, whose s is given.
// Either way the spans' first tiles follow each other, so a span's tiles are the difference to the next one's.
// More than kScanMax elements are not cut: a span each.
__device__ __forceinline__ void build_cut(const CutArgs &a, const CutLengths &raw, CutScratch &t, int w, int l)
{
    if (a.B > kScanMax) {
        for (int i = 64 * w + l; i < a.B; i += 64 * kCutWaves) {
            const int n = cut_length(a, a.lengths ? a.lengths[i] : a.n);
            a.spans[2 * i] = int4{i, 0, (n + 15) >> 4, i};
            a.spans[2 * i + 1] = int4{n, 16, 16, 16};
            a.pieces[i] = int2{i, 1};
        }
        return;
    }
    CutLengths len;                                          // (elements that do not exist: none)
#pragma unroll
    for (int c = 0; c < kCutMine; ++c) len.v[c] = 64 * (w + kCutWaves * c) + l < a.B ? cut_length(a, raw.v[c]) : 0;
    int end[kCutMine];                                       // tiles up to and including element i: in its chunk, then of all
#pragma unroll
    for (int c = 0; c < kCutMine; ++c) {
        end[c] = wave_scan((len.v[c] + 15) >> 4);
        if (l == 63) t.tiles[w + kCutWaves * c] = end[c];
    }
    __syncthreads();
    int total;
    {
        const int before = wave_scan(l < kCutChunks ? t.tiles[l] : 0);
        total = __builtin_amdgcn_readlane(before, kCutChunks - 1);
#pragma unroll
        for (int c = 0; c < kCutMine; ++c) {
            const int k = w + kCutWaves * c, i = 64 * k + l;
            if (k > 0) end[c] += __builtin_amdgcn_readlane(before, k - 1);
            if (i < a.B) { t.len[i] = len.v[c]; t.E[i + 1] = end[c]; }
        }
    }
    if (w == 0 && l == 0) t.E[0] = 0;
    if (w == 0 && l < 3) t.len[a.B + l] = 16;
    for (int g = 64 * w + l; g <= a.G; g += 64 * kCutWaves) t.first[g] = total;
    const int cspan = (total + a.kcost * a.B + a.G - 1) / a.G;

    // per element: sum_b ceil(tiles_b / s) is about total / s + B / 2; two guesses
    int s = a.short_tiles;
    const bool guesses = s == 0 && a.B > 1 && 2 * a.G > a.B;
    const int guess = guesses ? (2 * total + 2 * a.G - a.B - 1) / (2 * a.G - a.B) : 1;
    int spans_of[2][kCutMine];                               // spans up to and including element i, in its chunk
    if (s > 0) {                                             // (enough spans for it by the plan)
    } else if (a.B == 1) s = (total + a.G - 1) / a.G;
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const int sg = s > 0 ? s : guess + it * (1 + guess / 8);
        const float rs = 1.0f / (float)sg;
#pragma unroll
        for (int c = 0; c < kCutMine; ++c) {
            spans_of[it][c] = wave_scan(small_quotient(((len.v[c] + 15) >> 4) + sg - 1, sg, rs));
            if (l == 63) t.count[it][w + kCutWaves * c] = spans_of[it][c];
        }
    }
    __syncthreads();
    int runk[2];
#pragma unroll
    for (int it = 0; it < 2; ++it) runk[it] = wave_scan(l < kCutChunks ? t.count[it][l] : 0);
    int pick = 0;
    if (guesses) {
#pragma unroll
        for (int it = 1; it >= 0; --it) {                    // the smaller one, where both will do
            const int sg = guess + it * (1 + guess / 8);
            if (sg < cspan && __builtin_amdgcn_readlane(runk[it], kCutChunks - 1) <= a.G) { s = sg; pick = it; }
        }
    }
    if (s > 0) {
        const float rs = 1.0f / (float)s;
#pragma unroll
        for (int c = 0; c < kCutMine; ++c) {
            const int kk = w + kCutWaves * c;
            if (64 * kk >= a.B) continue;                    // uniform
            const int i = 64 * kk + l, tiles = (len.v[c] + 15) >> 4, k = small_quotient(tiles + s - 1, s, rs);
            const int before = kk == 0 ? 0 : pick ? __builtin_amdgcn_readlane(runk[1], max(kk - 1, 0)) : __builtin_amdgcn_readlane(runk[0], max(kk - 1, 0));
            const int last = before + (pick ? spans_of[1][c] : spans_of[0][c]);
            if (i < a.B) a.pieces[i] = int2{last - k, k};
            const int each = small_quotient(tiles, max(k, 1), 1.0f / (float)max(k, 1)), more = tiles - each * k;
            for (int j = 0; j < k; ++j) {                    // the k spans of an element differ by one tile at most
                t.first[last - k + j] = end[c] - tiles + j * each + min(j, more);
                t.owner[last - k + j] = i;
            }
        }
    } else {
        const float rc = 1.0f / (float)cspan;
#pragma unroll
        for (int c = 0; c < kCutMine; ++c) {
            const int i = 64 * (w + kCutWaves * c) + l, tiles = (len.v[c] + 15) >> 4;
            if (i >= a.B) continue;
            // this element's stretch of the axis, its gap included, is [x0, x1); spans that start in it
            const int x0 = end[c] - tiles + a.kcost * i, x1 = end[c] + a.kcost * (i + 1);
            for (int g = small_quotient(x0 + cspan - 1, cspan, rc); g * cspan < x1 && g < a.G; ++g) {
                t.first[g] = end[c] - tiles + max(g * cspan - x0 - a.kcost, 0);
                t.owner[g] = i;
            }
            const int g_lo = small_quotient(x0 + a.kcost, cspan, rc);
            a.pieces[i] = int2{g_lo + i, small_quotient(x1 - 1, cspan, rc) - g_lo + 1};
        }
    }
    __syncthreads();
    for (int g = 64 * w + l; g < a.G; g += 64 * kCutWaves) {
        const int t0 = t.first[g], tiles = t.first[g + 1] - t0;
        const int b = tiles > 0 ? t.owner[g] : 0;
        a.spans[2 * g] = int4{b, tiles > 0 ? t0 - t.E[b] : 0, tiles, s > 0 ? g : g + b};
        a.spans[2 * g + 1] = int4{t.len[b], t.len[b + 1], t.len[b + 2], t.len[b + 3]};
    }
}

} // namespace el
