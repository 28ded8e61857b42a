// The whole decode step (a1..a7 of Algorithm 3's attention routine) of a narrow fp32-arithmetic layer in ONE launch:
// one workgroup of eight wavefronts per batch element, every intermediate in LDS.
//
// At d_m = 64 or 128 a layer's four weight matrices are 64 or 256 KB: a workgroup can read all of them for itself, and
// does so before anything else (a wavefront keeps the fragments of its 16 output columns of every projection in
// registers, up to 128 of them).  As separate launches every step of the chain pays a launch and a round trip of its own.
// Bound: latency, of seven barriers and of the products between them (at d_m 128 also the 256 KB of weights through the compute unit's
// port).  Everything but W^O is under way before the first product, b^Q, c_out and the first positions of a5 included, which were
// fetched where they are used and waited for there (c_out between the stores of the result, one element after another); LDS operands
// are read together, and rows are reduced on the vector ALU instead of by twelve exchanges through LDS.  Per call among others, fp32:
// d_m 64, 2 sentences x 2 beams, n 32: 8.25 -> 6.6 us; 25 shapes of both widths 1.20 times as fast (1.02 to 1.30).  Arithmetic and
// rounding are those of generic_kernels.hip: fp32 operands, fp32 products and sums (16x16x4 MFMA), four consecutive k per lane.
#include <type_traits>
#include "mfma.h"

namespace el {

namespace {

constexpr int kSmallRows = 64;                          // heads * beam
constexpr int kSmallWork = 1 << 19;                     // padded rows x padded n x d_m (see small_step_applies)
constexpr int kSmallScores = kSmallWork / 64 + 4 * kSmallRows;      // floats of the score matrix, padded rows x (padded n + 4), at d_m >= 64

__device__ __forceinline__ f4 mfma4(float a, float b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f4 load4(const float *p) { return *(const f4 *)p; }
__device__ __forceinline__ f4 load4(const bf16_t *p)
{
    const u2 u = *(const u2 *)p;
    return f4{__uint_as_float(u[0] << 16), __uint_as_float(u[0] & 0xffff0000u), __uint_as_float(u[1] << 16), __uint_as_float(u[1] & 0xffff0000u)};
}
__device__ __forceinline__ f4 load4(const f16_t *p)
{
    const h4 h = *(const h4 *)p;
    return f4{(float)h[0], (float)h[1], (float)h[2], (float)h[3]};
}

// A sum of products in four chains, one per element of the fetched quads: in one chain the rounding errors of d_m additions
// pile up.  Error of the step against fp64 (relative 2-norm), one chain -> four: d_m 64 3.4e-7 -> 2.1e-7, d_m 128 5.0e-7 ->
// 2.7e-7 (a vector ALU kernel per step of the chain: 2.7e-7 and 4.1e-7).  Time unchanged.
struct Chains {
    f4 c[4];
    __device__ __forceinline__ Chains() { clear(); }
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int e = 0; e < 4; ++e) c[e] = f4{0.f, 0.f, 0.f, 0.f};
    }
    __device__ __forceinline__ void add(f4 a, f4 b)
    {
#pragma unroll
        for (int e = 0; e < 4; ++e) c[e] = mfma4(a[e], b[e], c[e]);
    }
    __device__ __forceinline__ f4 sum() const { return (c[0] + c[1]) + (c[2] + c[3]); }
};

// Over all 64 lanes on the vector ALU; every lane gets the result.
template <typename F>
__device__ __forceinline__ float over_wave(float v, F with)
{
    v = with(v, dpp<0xB1>(v)); v = with(v, dpp<0x4E>(v)); v = with(v, dpp<0x141>(v)); v = with(v, dpp<0x140>(v));
    const auto lane = [&](int i) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), i)); };
    return with(with(lane(0), lane(16)), with(lane(32), lane(48)));
}

struct SmallArgs {
    const void *H, *queries, *WqT, *Wk, *WvT, *WoT, *bq;
    const float *c_out;
    void *out;
    const int32_t *lengths;
    int64_t h_stride;
    int n, x, heads, d_k;
    float scale;
};

} // namespace

template <typename T, typename TO, int D>
__global__ void __launch_bounds__(512)
k_small_step(const SmallArgs a)
{
    constexpr int LD = D + 4;                           // row stride in LDS: 16 rows x 16 bytes reach all banks
    constexpr int KS = D / 16;                          // 16-wide slices of k; also 16-column blocks of a projection
    constexpr int CB = D / 64;
    __shared__ __attribute__((aligned(16))) float Qp[16 * LD];          // projected queries; later the head outputs A
    __shared__ __attribute__((aligned(16))) float Eq[kSmallRows * LD];  // expanded queries; later the weighted sums X
    __shared__ __attribute__((aligned(16))) float Sc[kSmallScores];     // scores, then probabilities
    __shared__ __attribute__((aligned(16))) float Pb[8 * 1024];         // partial weighted sums
    __shared__ float Li[kSmallRows];
    const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r16 = l & 15, q = l >> 4, b = blockIdx.x;
    const int x = a.x, R = a.heads * x, RT = (R + 15) >> 4;
    const bool mine = w < KS;                           // this wavefront has a block of projection columns: 16 w ..
    const int ncol = 16 * w + 4 * q;                    // a lane ends up with four consecutive columns of one row

    // the wavefront's share of a5: 16 rows x 64 columns, the positions split over the wavefronts that share a tile
    const int tiles = RT * CB, SP = 8 / tiles;          // RT <= 4, CB <= 2; SP is a power of two
    const bool sums = w < tiles * SP;
    const int tile5 = w % tiles, sp5 = w / tiles, rt5 = tile5 / CB, d5 = (tile5 - rt5 * CB) * 64;

    // Everything but W^O is requested before the first product, in straight code: what was fetched where it is used was waited for there,
    // and behind a branch the compiler lets a product wait for whatever the branch may have left out.
    f4 wq[KS], wk[KS], wv[KS], wo[KS], aq[KS], hf[KS], h5[2][4], bias_q, bias_out;
    int len = a.lengths ? a.lengths[b] : a.n;
    const T *Hb = (const T *)a.H + (size_t)b * a.h_stride;
    auto load_h = [&](int tt) __attribute__((always_inline)) {
        const T *hrow = Hb + (size_t)min(16 * tt + r16, len - 1) * D + 4 * q;
#pragma unroll
        for (int s = 0; s < KS; ++s) hf[s] = load4(hrow + 16 * s);
    };
    auto load_h5 = [&](int s0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                h5[u][j] = load4(Hb + (size_t)min(16 * (s0 + u * SP) + 4 * q + j, len - 1) * D + d5 + 4 * r16);
    };
    auto read_row = [](f4 (&v)[KS], const float *row) __attribute__((always_inline)) {     // all of it before the first product
#pragma unroll
        for (int s = 0; s < KS; ++s) v[s] = *(const f4 *)(row + 16 * s);
        __builtin_amdgcn_sched_barrier(0);
    };
    const size_t off = (size_t)(16 * (w % KS) + r16) * D + 4 * q;
    if (mine) {
        const T *qrow = (const T *)a.queries + ((size_t)b * x + min(r16, x - 1)) * D + 4 * q;
        bias_q = load4((const T *)(a.bq ? a.bq : a.WqT) + ncol);
#pragma unroll
        for (int s = 0; s < KS; ++s) { wq[s] = load4((const T *)a.WqT + off + 16 * s); aq[s] = load4(qrow + 16 * s); }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < KS; ++s) wk[s] = load4((const T *)a.Wk + off + 16 * s);
        __builtin_amdgcn_sched_barrier(0);
    }
    len = min(max(len, 1), a.n);                         // (the first thing that looks at it)
    const int tiles_t = (len + 15) >> 4, LS = 16 * tiles_t + 4;
    load_h(w / RT);                                      // (a wavefront without a tile of its own: a row that exists)
    load_h5(sp5);
    __builtin_amdgcn_sched_barrier(0);
    if (mine) {
#pragma unroll
        for (int s = 0; s < KS; ++s) wv[s] = load4((const T *)a.WvT + off + 16 * s);
        bias_out = load4(a.c_out + ncol);
        __builtin_amdgcn_sched_barrier(0);
        // a1
        Chains sums;
#pragma unroll
        for (int s = 0; s < KS; ++s) sums.add(wq[s], aq[s]);
        f4 acc = sums.sum();
        if (a.bq) acc += bias_q;
        *(f4 *)(Qp + r16 * LD + ncol) = acc * a.scale;
    }
    __syncthreads();
    // a2: head i contracts slices i d_k / 16 .. ; d_k is a multiple of 16
    if (mine) {
        Chains sums;
        int head = 0;
        f4 v[KS];
        read_row(v, Qp + r16 * LD + 4 * q);
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            sums.add(wk[s], v[s]);
            if (16 * (s + 1) % a.d_k == 0) {            // uniform
                if (r16 < x) *(f4 *)(Eq + (head * x + r16) * LD + ncol) = sums.sum();
                sums.clear();
                ++head;
            }
        }
        // (W^O into the registers that W^K has left; a3 to a6 hide its way)
#pragma unroll
        for (int s = 0; s < KS; ++s) wo[s] = load4((const T *)a.WoT + off + 16 * s);
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    // a3: tiles of 16 positions x 16 rows
    auto scores = [&](int tile) __attribute__((always_inline)) {
        const int tt = tile / RT, rt = tile - tt * RT;
        f4 v[KS];
        read_row(v, Eq + min(16 * rt + r16, R - 1) * LD + 4 * q);
        Chains sums;
#pragma unroll
        for (int s = 0; s < KS; ++s) sums.add(hf[s], v[s]);
        *(f4 *)(Sc + (16 * rt + r16) * LS + 16 * tt + 4 * q) = sums.sum();
    };
    if (w < tiles_t * RT) scores(w);
    for (int tile = w + 8; tile < tiles_t * RT; tile += 8) { load_h(tile / RT); scores(tile); }
    __syncthreads();
    // a4: a wavefront per row
    for (int r = w; r < R; r += 8) {
        float *row = Sc + r * LS;
        float m = -INFINITY, sum = 0.f;
        for (int t = l; t < len; t += 64) m = fmaxf(m, row[t]);
        m = over_wave(m, [](float x, float y) { return fmaxf(x, y); });
        for (int t = l; t < 16 * tiles_t; t += 64) {
            const float p = t < len ? expf(row[t] - m) : 0.f;
            sum += p;
            row[t] = p;
        }
        sum = over_wave(sum, [](float x, float y) { return x + y; });
        if (l == 0) Li[r] = sum;
    }
    __syncthreads();
    // a5
    if (sums) {
        f4 acc[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = f4{0.f, 0.f, 0.f, 0.f};
        auto sum = [&](int s0) __attribute__((always_inline)) {
            f4 p[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) p[u] = *(const f4 *)(Sc + min(16 * rt5 + r16, R - 1) * LS + 16 * min(s0 + u * SP, tiles_t - 1) + 4 * q);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (s0 + u * SP >= tiles_t) continue;    // uniform
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[e] = mfma4(p[u][j], h5[u][j][e], acc[e]);
            }
        };
        if (sp5 < tiles_t) sum(sp5);
        for (int s0 = sp5 + 2 * SP; s0 < tiles_t; s0 += 2 * SP) { load_h5(s0); sum(s0); }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *(f4 *)(Pb + ((w * 16) + 4 * q + i) * 64 + 4 * r16) = f4{acc[0][i], acc[1][i], acc[2][i], acc[3][i]};
    }
    __syncthreads();
    auto add_up = [&](auto count) __attribute__((always_inline)) {
        constexpr int C = decltype(count)::value;
        for (int i = threadIdx.x; i < tiles * 256; i += 512) {
            const int tile = i >> 8, row = (i >> 4) & 15, quad = i & 15, rt = tile / CB, r = 16 * rt + row;
            if (r >= R) continue;
            f4 part[C], v = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int sp = 0; sp < C; ++sp) part[sp] = *(const f4 *)(Pb + ((sp * tiles + tile) * 16 + row) * 64 + 4 * quad);
            const float li = Li[r];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int sp = 0; sp < C; ++sp) v += part[sp];
            *(f4 *)(Eq + r * LD + (tile - rt * CB) * 64 + 4 * quad) = v / li;
        }
    };
    const int parts = min(SP, tiles_t);                  // the wavefronts beyond have no positions: zeros
    if (parts > 4) add_up(std::integral_constant<int, 8>{});
    else if (parts > 2) add_up(std::integral_constant<int, 4>{});
    else if (parts > 1) add_up(std::integral_constant<int, 2>{});
    else add_up(std::integral_constant<int, 1>{});
    __syncthreads();
    // a6: the 16 columns of a wavefront belong to one head
    if (mine) {
        const int head = 16 * w / a.d_k;
        f4 v[KS];
        read_row(v, Eq + (head * x + min(r16, x - 1)) * LD + 4 * q);
        Chains sums;
#pragma unroll
        for (int s = 0; s < KS; ++s) sums.add(wv[s], v[s]);
        *(f4 *)(Qp + r16 * LD + ncol) = sums.sum();
    }
    __syncthreads();
    // a7
    if (mine) {
        f4 v[KS];
        read_row(v, Qp + r16 * LD + 4 * q);
        Chains sums;
#pragma unroll
        for (int s = 0; s < KS; ++s) sums.add(wo[s], v[s]);
        const f4 acc = sums.sum() + bias_out;
        if (r16 < x) {
            TO *o = (TO *)a.out + ((size_t)b * x + r16) * D + ncol;
#pragma unroll
            for (int e = 0; e < 4; ++e) from_f32(acc[e], o + e);
        }
    }
}

// Where one workgroup per batch element does the whole step: the weights fit its registers (d_m 64 or 128, head sizes that
// are whole 16-wide slices), at most 16 beams (one row tile), and its scores and weighted sums, R x n x d_m products each on
// one compute unit, stay below what the separate launches need for their extra round trips.  us, here against separately (up to 16
// elements the separate side is the host's 22 us for six launches where it takes longer than the device):
//                                        1 element    16           256          1024         4096
//   d_m 64, 4 heads, 2 beams, n 32       6.3 / 22.1   6.6 / 23.1   6.9 / 22.5   23.5 / 33.2  91.9 / 91.5
//   d_m 64, 4 heads, 16 beams, n 64      12.0 / 22.2  12.4 / 23.0  12.7 / 38.4  46.9 / 112   184 / 402
//   d_m 128, 2 heads, 4 beams, n 100     15.8 / 22.0  16.1 / 23.2  16.5 / 30.6  62.0 / 72.2  244 / 247
//   d_m 128, 2 heads, 4 beams, n 256     20.0 / 21.7  20.4 / 22.7  21.2 / 38.1  82.3 / 102   330 / 392     2^19
//   d_m 128, 8 heads, 8 beams, n 64      23.6 / 18.2  24.1 / 19.2  24.8 / 60.8  95.3 / 188   378 / 746     2^19
// and 25.5 / 18.6 at 2^20 (d_m 64, 64 rows, n 256, 2 elements).  So the line is right for a batch and generous for a few
// elements near it; thousands of elements of few rows come out even, because beyond one element per
// compute unit the workgroups run in rounds that each read the weights again.
bool small_step_applies(const Problem &p)
{
    if ((p.d_m != 64 && p.d_m != 128) || p.d_k % 16 != 0 || p.beam > 16 || p.R > kSmallRows) return false;
    const int64_t n16 = (p.n + 15) / 16 * 16, r16 = (p.R + 15) / 16 * 16;
    if (r16 * n16 * p.d_m > kSmallWork) return false;
    const size_t four = 4 * dtype_size(p.dtype);         // operands are fetched four elements at a time
    return p.H_batch_stride % 4 == 0 && ((uintptr_t)p.H & (four - 1)) == 0 && ((uintptr_t)p.queries & (four - 1)) == 0;
}

template <typename T, typename TO>
static void launch_small_t(const SmallArgs &a, int d_m, int B, hipStream_t s)
{
    if (d_m == 64) hipLaunchKernelGGL((k_small_step<T, TO, 64>), dim3(B), dim3(512), 0, s, a);
    else hipLaunchKernelGGL((k_small_step<T, TO, 128>), dim3(B), dim3(512), 0, s, a);
}

hipError_t launch_small_step(const el_attn_ctx *ctx, const Problem &p, hipStream_t s)
{
    SmallArgs a;
    a.H = p.H; a.queries = p.queries; a.WqT = ctx->w.WqT; a.Wk = ctx->w.Wk; a.WvT = ctx->w.WvTs; a.WoT = ctx->w.WoTs; a.bq = ctx->w.bq;
    a.c_out = ctx->w.c_out; a.out = p.out; a.lengths = p.lengths; a.h_stride = p.H_batch_stride;
    a.n = p.n; a.x = p.beam; a.heads = p.heads; a.d_k = p.d_k;
    a.scale = 1.0f / sqrtf((float)p.d_k);
    const bool f32_out = p.out_dtype == EL_F32;
    if (p.dtype == EL_F32) launch_small_t<float, float>(a, p.d_m, p.B, s);
    else if (p.dtype == EL_F16) { if (f32_out) launch_small_t<f16_t, float>(a, p.d_m, p.B, s); else launch_small_t<f16_t, f16_t>(a, p.d_m, p.B, s); }
    else { if (f32_out) launch_small_t<bf16_t, float>(a, p.d_m, p.B, s); else launch_small_t<bf16_t, bf16_t>(a, p.d_m, p.B, s); }
    return hipGetLastError();
}

} // namespace el
