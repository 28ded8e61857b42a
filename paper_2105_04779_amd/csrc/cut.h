// How the attention core's work is cut, worked out on the device from the actual lengths by ONE wavefront: a table of
// spans (what each workgroup of the core walks) and a table of pieces (where the partial results of a batch element
// are), both read with one load.  The wavefront rides in the launch that precedes the core (k_qelq), under that
// kernel's memory latency: in the core, every workgroup repeated the scan of all lengths (1.7 us of every launch at
// 64 batch elements) before it could request its first tile.  Everything is element- or span-parallel over the lanes, with
// no dependent chain through LDS beyond one write and one read.
#pragma once
#include "el_internal.h"

namespace el {

constexpr int kCutChunks = kScanMax / 64;

// LDS of the one wavefront: prefix of tiles, lengths, and per span its first tile and its element
struct CutScratch { int E[kScanMax + 1], len[kScanMax + 3], first[kSpanMax + 1], owner[kSpanMax]; };
struct CutLengths { int v[kCutChunks]; };            // lane l: lengths of elements l, 64 + l, ...

__device__ __forceinline__ int cut_length(const CutArgs &a, int i) { return a.lengths ? min(max(a.lengths[i], 1), a.n) : a.n; }

// All lengths requested at once, and ahead of whatever else the wavefront has to fetch.
__device__ __forceinline__ void load_cut_lengths(const CutArgs &a, int l, CutLengths &t)
{
#pragma unroll
    for (int c = 0; c < kCutChunks; ++c) t.v[c] = a.B <= kScanMax && 64 * c + l < a.B ? cut_length(a, 64 * c + l) : 0;
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

// Executed by one wavefront (lane l).  Two ways to cut, the one with the shorter longest span wins:
//   flattened   the 16-row tiles of all elements lie on one axis, element after element, each element preceded by a
//               gap of `kcost` units (what moving on to a new element costs a workgroup, in tiles): tile kt of element
//               b sits at E[b] + kcost (b + 1) + kt.  The axis is cut into G equal spans; span g's piece of element b
//               is slot g + b (unique: along the axis, span and element never decrease and one of them grows).
//   per element every element is cut into its own spans of at most s tiles: nothing crosses, a piece is a span and has
//               its number.  The better one for few elements (one sentence: the flattened axis would start with a gap
//               for nothing), and the only one for the core of short spans, whose s is given.
// Either way the spans' first tiles follow each other, so a span's tiles are the difference to the next one's.
// More than kScanMax elements are not cut: a span each.
__device__ __forceinline__ void build_cut(const CutArgs &a, const CutLengths &len, CutScratch &t, int l)
{
    if (a.B > kScanMax) {
        for (int i = l; i < a.B; i += 64) {
            const int n = cut_length(a, i);
            a.spans[2 * i] = int4{i, 0, (n + 15) >> 4, i};
            a.spans[2 * i + 1] = int4{n, 16, 16, 16};
            a.pieces[i] = int2{i, 1};
        }
        return;
    }
    int end[kCutChunks], total = 0;                          // tiles of elements 0 .. i
#pragma unroll
    for (int c = 0; c < kCutChunks; ++c) {
        end[c] = total;
        if (64 * c >= a.B) continue;                         // uniform
        const int i = 64 * c + l;
        end[c] = total + wave_scan((len.v[c] + 15) >> 4);
        total = __builtin_amdgcn_readlane(end[c], 63);
        if (i < a.B) { t.len[i] = len.v[c]; t.E[i + 1] = end[c]; }
    }
    if (l == 0) t.E[0] = 0;
    if (l < 3) t.len[a.B + l] = 16;
    for (int g = l; g <= a.G; g += 64) t.first[g] = total;
    __builtin_amdgcn_wave_barrier();
    const int cspan = (total + a.kcost * a.B + a.G - 1) / a.G;

    // per element: sum_b ceil(tiles_b / s) is about total / s + B / 2; two guesses
    int s = a.short_tiles;
    if (s > 0) {                                             // (enough spans for it by the plan)
    } else if (a.B == 1) s = (total + a.G - 1) / a.G;
    else if (2 * a.G > a.B) {
        const int guess = (2 * total + 2 * a.G - a.B - 1) / (2 * a.G - a.B);
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const int sg = guess + it * (1 + guess / 8);
            if (s > 0 || sg >= cspan) continue;              // uniform
            const float rs = 1.0f / (float)sg;
            int cnt = 0;
#pragma unroll
            for (int c = 0; c < kCutChunks; ++c) {
                if (64 * c >= a.B) continue;
                cnt += small_quotient(((len.v[c] + 15) >> 4) + sg - 1, sg, rs);
            }
            if (__builtin_amdgcn_readlane(wave_scan(cnt), 63) <= a.G) s = sg;
        }
    }
    if (s > 0) {
        int runk = 0;
        const float rs = 1.0f / (float)s;
#pragma unroll
        for (int c = 0; c < kCutChunks; ++c) {
            if (64 * c >= a.B) continue;
            const int i = 64 * c + l, tiles = (len.v[c] + 15) >> 4, k = small_quotient(tiles + s - 1, s, rs), last = runk + wave_scan(k);
            if (i < a.B) a.pieces[i] = int2{last - k, k};
            const int each = small_quotient(tiles, max(k, 1), 1.0f / (float)max(k, 1)), more = tiles - each * k;
            for (int j = 0; j < k; ++j) {                    // the k spans of an element differ by one tile at most
                t.first[last - k + j] = end[c] - tiles + j * each + min(j, more);
                t.owner[last - k + j] = i;
            }
            runk = __builtin_amdgcn_readlane(last, 63);
        }
    } else {
        const float rc = 1.0f / (float)cspan;
#pragma unroll
        for (int c = 0; c < kCutChunks; ++c) {
            if (64 * c >= a.B) continue;
            const int i = 64 * c + l, tiles = (len.v[c] + 15) >> 4;
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
    __builtin_amdgcn_wave_barrier();
    for (int g = l; g < a.G; g += 64) {
        const int t0 = t.first[g], tiles = t.first[g + 1] - t0;
        const int b = tiles > 0 ? t.owner[g] : 0;
        a.spans[2 * g] = int4{b, tiles > 0 ? t0 - t.E[b] : 0, tiles, s > 0 ? g : g + b};
        a.spans[2 * g + 1] = int4{t.len[b], t.len[b + 1], t.len[b + 2], t.len[b + 3]};
    }
}

} // namespace el
