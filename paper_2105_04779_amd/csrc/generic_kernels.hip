// fp32-arithmetic kernels for every step of the EL-attention decode step.
//
// They cover every dtype and shape (the fp32 configuration runs on them alone) and are the fallback wherever
// no 16-bit MFMA kernel applies.  Storage values are widened exactly and every product and sum is fp32: the
// contractions run on the fp32 matrix instruction (16x16x4: fp32 operands, fp32 accumulators, 64 FLOP a clock
// and SIMD, twice the vector ALU without its operand traffic).  Weights are stored transposed at prepare time,
// so every operand is contiguous along the contraction and a lane fetches four consecutive k at once: step j of
// four instructions then contracts k = 16 s + 4 g + j over the lane groups g, the same permutation on both sides.
//
// Steps follow Algorithm 3's attention routine (appendix A) and Eq. 5 / Eq. 9:
//   qproj  a1  Qp = (q W^Q + b^Q) / sqrt(d_k)
//   elq    a2  EL-Q_i = Qp_i (W_i^K)^T                      rows r = i*beam + j
//   core   a3-a5  scores against H (k_gemm_f32 per batch element), softmax over the valid prefix and weighted
//                 sum of H (k_sum_f32)
//   vproj  a6  A_i = X_i W_i^V
//   oproj  a7  out = A W^O + c_out,  c_out = b^O + sum_i b_i^V W_i^O (Eq. 8/9)
#include <type_traits>
#include "el_internal.h"

namespace el {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned int u2v __attribute__((ext_vector_type(2)));

constexpr int kBlock = 256;
constexpr int kGemmWaves = 8;
constexpr int kChunk = 512; // key positions scored per pass of k_core_generic and of k_sum_f32

static inline int cdiv(int a, int b) { return (a + b - 1) / b; }

__device__ __forceinline__ f4 mfma4(float a, float b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// four consecutive elements, widened
__device__ __forceinline__ f4 load4(const float *p) { return *(const f4 *)p; }
__device__ __forceinline__ f4 load4(const bf16_t *p)
{
    const u2v u = *(const u2v *)p;
    return f4{__uint_as_float(u[0] << 16), __uint_as_float(u[0] & 0xffff0000u), __uint_as_float(u[1] << 16), __uint_as_float(u[1] & 0xffff0000u)};
}
__device__ __forceinline__ f4 load4(const f16_t *p)
{
    typedef _Float16 h4 __attribute__((ext_vector_type(4)));
    const h4 h = *(const h4 *)p;
    return f4{(float)h[0], (float)h[1], (float)h[2], (float)h[3]};
}
// elements k .. k + 3 of a row of K, zero where they do not exist.  VEC: K and the row's address are multiples of four elements.
template <bool VEC, typename T>
__device__ __forceinline__ f4 load_k4(const T *row, int k, int K)
{
    if (VEC) { if (k < K) return load4(row + k); return f4{0.f, 0.f, 0.f, 0.f}; }
    f4 v = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (k + e < K) v[e] = to_f32(row[k + e]);
    return v;
}
template <bool VEC, typename T>
__device__ __forceinline__ f4 load_full4(const T *p)
{
    if (VEC) return load4(p);
    return f4{to_f32(p[0]), to_f32(p[1]), to_f32(p[2]), to_f32(p[3])};
}

// ---------------------------------------------------------------------------------------------
// c_out[d] = b^O[d] + sum_c b^V[c] W^O[c, d]: a wavefront per output, W^O transposed.
template <typename T>
__global__ void __launch_bounds__(kBlock)
k_cout(const T *__restrict__ bv, const T *__restrict__ bo, const T *__restrict__ WoT, float *__restrict__ c_out, int hd, int d_m)
{
    const int d = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6), l = threadIdx.x & 63;
    if (d >= d_m) return;
    float acc = 0.f;
    if (bv)
        for (int c = l; c < hd; c += 64) acc = fmaf(to_f32(bv[c]), to_f32(WoT[(size_t)d * hd + c]), acc);
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    if (l == 0) c_out[d] = acc + (bo ? to_f32(bo[d]) : 0.f);
}

// ---------------------------------------------------------------------------------------------
// C[m, n] = (sum_k A[m, k] Bt[n, k] + bias[n]) * scale, batched over z (a head, or a batch element for the
// scores).  One workgroup owns (16 MT) x (16 NT) outputs; its eight wavefronts each take an eighth of k straight from
// global memory into registers (consecutive slices, so both halves of a cache line go to one wavefront), four
// 16-wide slices of both operands requested before the first is used (up to K = 512 the whole contraction is one
// round trip), and add up through LDS.
// Bound: memory latency at decode batch sizes, the fp32 matrix rate beyond.
// 64 x 512 x 512: 4.6 us, 119 us for the kernel it replaces (one output per thread, a serial loop over k); the
// scores of 16 x 32 rows over 300 positions, K = 512: 8.9 us.
// Three forms (launch_gemm_f32 has the rule):
//   early     what needs neither the length nor the sums is requested before either is waited for: bias, then rows, then the length's
//             operand; groups of four slices in straight code, so that the first products wait for their own operands and not for the
//             last ones.  With the bias fetched behind the last barrier, element by element, and everything behind the length: 64 x
//             512 x 512 with a bias 5.5 -> 4.6 us, the scores above 9.4 -> 8.9.  Rows held across the wait for the length take 66
//             registers instead of 49 (16 x 16 outputs), 104 instead of 68 (32 x 16): a workgroup less on a compute unit.
//   straight  the groups in straight code, everything behind the length
//   branched  every slice behind its own branch, the bias behind the last products: the fewest instructions
enum GemmForm { kGemmEarly, kGemmStraight, kGemmBranched };
struct GemmF32 {
    const void *A, *Bt;
    void *C;
    const void *bias;        // storage type, may be null
    const float *bias32;     // may be null
    const int32_t *lengths;  // scores: valid rows of Bt of element z (null elsewhere or: all N)
    float scale;
    int M, N, K;
    int64_t lda, ldb, ldc;
    int64_t za, zb, zc;      // element offsets per z
    int x, R;                // for the row maps: logical row m of head z is row (m / x) R + z x + m % x
    int map_a, map_c;
    int use_lengths, vec_c;
};

template <typename TA, typename TB, typename TO, bool VEC, int MT, int NT, GemmForm FORM>
__global__ void __launch_bounds__(64 * kGemmWaves)
k_gemm_f32(const GemmF32 g)
{
    constexpr int NW = kGemmWaves, U = 4;
    constexpr bool EARLY = FORM == kGemmEarly;
    __shared__ f4 red[NW * MT * NT * 64];
    const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r16 = l & 15, q = l >> 4, z = blockIdx.z;
    const int n0 = blockIdx.x * (16 * NT), m0 = blockIdx.y * (16 * MT);
    int N = g.N;
    if (EARLY) {
        if (g.use_lengths && g.lengths) N = g.lengths[z];     // (looked at below)
    } else if (g.use_lengths) {
        if (g.lengths) N = min(max(g.lengths[z], 1), N);
        if (n0 >= N) return;
    }
    auto mapped = [&](int m) -> int64_t { return (int64_t)(m / g.x) * g.R + (int64_t)z * g.x + m % g.x; };
    const TA *ap[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        const int m = min(m0 + 16 * i + r16, g.M - 1);
        ap[i] = (const TA *)g.A + (g.map_a ? mapped(m) : (int64_t)m) * g.lda + z * g.za + 4 * q;
    }
    const int full = g.K >> 4, per = (full + NW - 1) / NW, s_begin = w * per, s_end = min(full, (w + 1) * per);
    f4 first[U][MT], bias = f4{0.f, 0.f, 0.f, 0.f};
    // (WHOLE: all U slices of the group exist)
    auto load_first = [&](auto whole, int s0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (!decltype(whole)::value && s0 + u >= s_end) continue;      // uniform
#pragma unroll
            for (int i = 0; i < MT; ++i) first[u][i] = load_full4<VEC>(ap[i] + 16 * (s0 + u));
        }
    };
    // (the bias in two places, written out: as a lambda it has the compiler fetch the arguments one by one, each waited for)
    if (EARLY && w < MT * NT) {                                    // the wavefront that adds a tile up
        const int n = n0 + 16 * (w % NT) + 4 * q;
        if (g.bias) {
#pragma unroll
            for (int e = 0; e < 4; ++e) bias[e] = to_f32(((const TB *)g.bias)[min(n + e, g.N - 1)]);
        } else if (g.bias32) {
#pragma unroll
            for (int e = 0; e < 4; ++e) bias[e] = g.bias32[min(n + e, g.N - 1)];
        }
    }
    if (EARLY) {
        if (s_begin + U <= s_end) load_first(std::true_type{}, s_begin);
        else load_first(std::false_type{}, s_begin);
        asm volatile("" ::: "memory");                        // (requested here, not behind the wait for the length)
        if (g.use_lengths) {
            N = min(max(N, 1), g.N);
            if (n0 >= N) return;
        }
    }
    const TB *bp[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) bp[j] = (const TB *)g.Bt + (int64_t)min(n0 + 16 * j + r16, N - 1) * g.ldb + z * g.zb + 4 * q;

    f4 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
    // weights (or H) as the instruction's A operand: a lane ends up with four consecutive n of one m
    auto product = [&](const f4 *a, const f4 *b) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j) acc[i][j] = mfma4(b[j][e], a[i][e], acc[i][j]);
    };
    // Where in the instruction stream a group starts: 16 bytes past a multiple of 32.  At a multiple of 32, which is where it may land with
    // whatever comes before it, 32 x 32 outputs take 1.09 times as long (1024 rows, K = 512, 512 columns: 13.4 against 12.3 us).
    auto place = [&]() __attribute__((always_inline)) {
        if (MT > 1) asm volatile(".p2align 5\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0");
    };
    if constexpr (FORM == kGemmBranched) {
        for (int s0 = s_begin; s0 < s_end; s0 += U) {
            f4 a[U][MT], b[U][NT];
            place();
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (s0 + u >= s_end) continue;                // uniform
#pragma unroll
                for (int i = 0; i < MT; ++i) a[u][i] = load_full4<VEC>(ap[i] + 16 * (s0 + u));
#pragma unroll
                for (int j = 0; j < NT; ++j) b[u][j] = load_full4<VEC>(bp[j] + 16 * (s0 + u));
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (s0 + u >= s_end) continue;
                product(a[u], b[u]);
            }
        }
    } else {
        auto group = [&](auto whole, int s0) __attribute__((always_inline)) {
            f4 a[U][MT], b[U][NT];
            if (!EARLY) place();
            else if (s0 > s_begin) load_first(whole, s0);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (!decltype(whole)::value && s0 + u >= s_end) continue;
                if (!EARLY)
#pragma unroll
                    for (int i = 0; i < MT; ++i) a[u][i] = load_full4<VEC>(ap[i] + 16 * (s0 + u));
#pragma unroll
                for (int j = 0; j < NT; ++j) b[u][j] = load_full4<VEC>(bp[j] + 16 * (s0 + u));
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (!decltype(whole)::value && s0 + u >= s_end) continue;
                product(EARLY ? first[u] : a[u], b[u]);
            }
        };
        for (int s0 = s_begin; s0 < s_end; s0 += U) {
            if (s0 + U <= s_end) group(std::true_type{}, s0);
            else group(std::false_type{}, s0);
        }
    }
    if ((g.K & 15) && w == NW - 1) {                          // the slice that is not full
        f4 at[MT], b[NT];
#pragma unroll
        for (int i = 0; i < MT; ++i) at[i] = load_k4<VEC>(ap[i] - 4 * q, 16 * full + 4 * q, g.K);
#pragma unroll
        for (int j = 0; j < NT; ++j) b[j] = load_k4<VEC>(bp[j] - 4 * q, 16 * full + 4 * q, g.K);
        product(at, b);
    }
    if (!EARLY && w < MT * NT) {
        const int n = n0 + 16 * (w % NT) + 4 * q;
        if (g.bias) {
#pragma unroll
            for (int e = 0; e < 4; ++e) bias[e] = to_f32(((const TB *)g.bias)[min(n + e, g.N - 1)]);
        } else if (g.bias32) {
#pragma unroll
            for (int e = 0; e < 4; ++e) bias[e] = g.bias32[min(n + e, g.N - 1)];
        }
    }
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) red[(w * MT * NT + i * NT + j) * 64 + l] = acc[i][j];
    __syncthreads();
    static_assert(MT * NT <= NW, "a tile per wavefront");
    if (w < MT * NT) {
        const int tile = w;
        f4 v = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < NW; ++s) v += red[(s * MT * NT + tile) * 64 + l];
        const int m = m0 + 16 * (tile / NT) + r16, n = n0 + 16 * (tile % NT) + 4 * q;
        if (m >= g.M) return;
        TO *c = (TO *)g.C + (g.map_c ? mapped(m) : (int64_t)m) * g.ldc + z * g.zc + n;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (g.bias || g.bias32) v[e] += bias[e];
            v[e] *= g.scale;
        }
        if (sizeof(TO) == 4 && g.vec_c && n + 4 <= N) *(f4 *)c = v;
        else
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (n + e < N) from_f32(v[e], c + e);
    }
}

// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ float wave_sum(float v)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ float wave_max(float v)
{
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

// a4 + a5: softmax of the scores S [B, R, ldS] over the valid prefix and the weighted sum of H, normalised:
// Xn[b, r, d0 .. d0 + 63] for 16 rows r.  Every workgroup works its 16 rows' probabilities out for itself (R n
// exponentials against the R n d_m / 8 products of a 64-column block) and keeps them in LDS, 512 positions at a
// time; the wavefronts take every eighth 16-position slice.  The scores and the first slices of H are requested
// together, before anything waits.  A lane fetches four consecutive columns of one row of H, so a load instruction
// reads 4 rows x 256 contiguous bytes, and column c of the block is column c / 4 of accumulator c % 4.  Bound: memory
// latency, then the fp32 matrix rate.  16 x 32 rows, 300 positions, d_m 512: 7.6 us; with the scores (above) 16.5 us
// against the 125 us of the kernels with one row per workgroup and their merge.
template <typename T, bool VEC>
__global__ void __launch_bounds__(512)
k_sum_f32(const float *__restrict__ S, int64_t ldS, const T *__restrict__ H, int64_t h_stride, const int32_t *__restrict__ lengths,
          int n, int d_m, int R, float *__restrict__ Xn, float *__restrict__ ML)
{
    constexpr int NW = 8, RW = 16 / NW, PS = kChunk + 4, U = 4, PL = kChunk / 64;
    __shared__ __attribute__((aligned(16))) float Ps[16 * PS];
    __shared__ float Li[16];
    const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r16 = l & 15, q = l >> 4;
    const int d0 = blockIdx.x * 64, r0 = blockIdx.y * 16, b = blockIdx.z;
    int len = lengths ? lengths[b] : n;                       // (looked at behind the scores' requests)
    const T *Hb = H + (size_t)b * h_stride;
    const float *srow[RW];
#pragma unroll
    for (int i = 0; i < RW; ++i) srow[i] = S + ((size_t)b * R + min(r0 + RW * w + i, R - 1)) * ldS;
    // the scores of one chunk of this wavefront's rows, all requested together and without regard to the length (a row of S has n
    // values; what is past the length is whatever the workspace holds, and masked before it is looked at)
    float sv[RW][PL];
    auto load_scores = [&](int c0) {
#pragma unroll
        for (int k = 0; k < PL; ++k)
#pragma unroll
            for (int i = 0; i < RW; ++i) {
                sv[i][k] = -INFINITY;
                if (c0 + 64 * k < n) sv[i][k] = srow[i][min(c0 + 64 * k + l, n - 1)];        // (uniform)
            }
    };
    auto mask_scores = [&](int c0) {
#pragma unroll
        for (int i = 0; i < RW; ++i)
#pragma unroll
            for (int k = 0; k < PL; ++k) sv[i][k] = c0 + 64 * k + l < len ? sv[i][k] : -INFINITY;
    };
    // a slice of H per wavefront in flight: U slices of 16 positions
    const int col = d0 + 4 * r16;
    f4 h[U][4];
    auto load_h = [&](int c0, int s0, int slices) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (s0 + NW * u >= slices) continue;               // uniform
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                // a position that does not exist has probability zero: any valid row stands in for it
                const int t = min(c0 + 16 * (s0 + NW * u) + 4 * q + j, len - 1);
                h[u][j] = load_k4<VEC>(Hb + (size_t)t * d_m, col, d_m);
            }
        }
    };
    load_scores(0);
    asm volatile("" ::: "memory");                            // (requested here, not behind the wait for the length)
    len = min(max(len, 1), n);
    load_h(0, w, (min(kChunk, len) + 15) >> 4);
    float mx[RW], sum[RW];
#pragma unroll
    for (int i = 0; i < RW; ++i) { mx[i] = -INFINITY; sum[i] = 0.f; }
    auto fold_max = [&]() {
#pragma unroll
        for (int i = 0; i < RW; ++i)
#pragma unroll
            for (int k = 0; k < PL; ++k) mx[i] = fmaxf(mx[i], sv[i][k]);
    };
    mask_scores(0);
    fold_max();
    if (len > kChunk) {
        for (int c0 = kChunk; c0 < len; c0 += kChunk) { load_scores(c0); mask_scores(c0); fold_max(); }
        load_scores(0);
        mask_scores(0);
    }
#pragma unroll
    for (int i = 0; i < RW; ++i) mx[i] = wave_max(mx[i]);
    f4 acc[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] = f4{0.f, 0.f, 0.f, 0.f};
    for (int c0 = 0; c0 < len; c0 += kChunk) {
        const int slices = (min(kChunk, len - c0) + 15) >> 4;
        if (c0 > 0) __syncthreads();
#pragma unroll
        for (int i = 0; i < RW; ++i)
#pragma unroll
            for (int k = 0; k < PL; ++k) {
                const float p = expf(sv[i][k] - mx[i]);       // zero where the position does not exist
                sum[i] += p;
                Ps[(RW * w + i) * PS + 64 * k + l] = p;
            }
        __syncthreads();
        if (c0 + kChunk < len) { load_scores(c0 + kChunk); mask_scores(c0 + kChunk); }
        for (int s0 = w; s0 < slices; s0 += NW * U) {
            if (c0 > 0 || s0 > w) load_h(c0, s0, slices);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (s0 + NW * u >= slices) continue;
                const f4 p = *(const f4 *)(Ps + r16 * PS + 16 * (s0 + NW * u) + 4 * q);
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[e] = mfma4(p[j], h[u][j][e], acc[e]);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        const float s = wave_sum(sum[i]);
        const int r = r0 + RW * w + i;
        if (l == 0) {
            Li[RW * w + i] = s;
            if (d0 == 0 && r < R) { ML[((size_t)b * R + r) * 2] = mx[i]; ML[((size_t)b * R + r) * 2 + 1] = s; }
        }
    }
    __syncthreads();                                          // the probabilities are no longer needed
    f4 *red = (f4 *)Ps;                                       // [wavefront][row][16 quads]
#pragma unroll
    for (int i = 0; i < 4; ++i) red[(w * 16 + 4 * q + i) * 16 + r16] = f4{acc[0][i], acc[1][i], acc[2][i], acc[3][i]};
    __syncthreads();
    const int row = threadIdx.x >> 4, quad = threadIdx.x & 15, d = d0 + 4 * quad;
    if (row >= 16 || r0 + row >= R) return;
    f4 v = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NW; ++s) v += red[(s * 16 + row) * 16 + quad];
    const float inv = Li[row];
    float *xo = Xn + ((size_t)b * R + r0 + row) * d_m + d;
    if (VEC) {                                                // (d_m is a multiple of four)
        if (d < d_m) *(f4 *)xo = f4{v[0] / inv, v[1] / inv, v[2] / inv, v[3] / inv};
    } else
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (d + e < d_m) xo[e] = v[e] / inv;
}

// ---------------------------------------------------------------------------------------------
// a3-a5 without scores in memory, for keys so long next to d_m that the scores do not fit the workspace (see scores_fit):
// one (row r, key-range part p, batch element b) per workgroup, on the vector ALU.
// Writes the un-normalised weighted sum, and the running max / sum of its range.
template <typename T, int MAXD>
__global__ void __launch_bounds__(kBlock)
k_core_generic(const float *__restrict__ elq, const T *__restrict__ H, int64_t h_stride,
               const int32_t *__restrict__ lengths, int n, int d_m, int R, int Rstride, int parts,
               float *__restrict__ Xp, float *__restrict__ ML)
{
    extern __shared__ float smem[];
    float *q_s = smem;          // [d_m]
    float *s_s = smem + d_m;    // [kChunk]
    __shared__ float red[8];

    const int r = blockIdx.x, p = blockIdx.y, b = blockIdx.z;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int len = lengths ? lengths[b] : n;
    len = min(max(len, 1), n);
    const int t0 = (int)(((int64_t)len * p) / parts);
    const int t1 = (int)(((int64_t)len * (p + 1)) / parts);
    const T *Hb = H + (size_t)b * h_stride;

    for (int d = tid; d < d_m; d += kBlock) q_s[d] = elq[((size_t)b * R + r) * d_m + d];
    __syncthreads();

    float m = -INFINITY, l = 0.f;
    float acc[MAXD];
#pragma unroll
    for (int k = 0; k < MAXD; ++k) acc[k] = 0.f;

    for (int c0 = t0; c0 < t1; c0 += kChunk) {
        const int cnt = min(kChunk, t1 - c0);
        // scores of this chunk: one wave per key position, lanes over d
        for (int t = wave; t < cnt; t += kBlock / 64) {
            const T *hr = Hb + (size_t)(c0 + t) * d_m;
            float dot = 0.f;
            for (int d = lane; d < d_m; d += 64) dot = fmaf(q_s[d], to_f32(hr[d]), dot);
            dot = wave_sum(dot);
            if (lane == 0) s_s[t] = dot;
        }
        __syncthreads();
        float cm = -INFINITY;
        for (int t = tid; t < cnt; t += kBlock) cm = fmaxf(cm, s_s[t]);
        cm = wave_max(cm);
        if (lane == 0) red[wave] = cm;
        __syncthreads();
        cm = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
        const float m_new = fmaxf(m, cm);
        const float alpha = (m == -INFINITY) ? 0.f : expf(m - m_new);
        float ps = 0.f;
        for (int t = tid; t < cnt; t += kBlock) {
            float e = expf(s_s[t] - m_new);
            s_s[t] = e;
            ps += e;
        }
        ps = wave_sum(ps);
        if (lane == 0) red[4 + wave] = ps;
        __syncthreads();
        l = l * alpha + (red[4] + red[5] + red[6] + red[7]);
        m = m_new;
#pragma unroll
        for (int k = 0; k < MAXD; ++k) {
            const int d = tid + k * kBlock;
            if (d < d_m) {
                float a = acc[k] * alpha;
                for (int t = 0; t < cnt; ++t) a = fmaf(s_s[t], to_f32(Hb[(size_t)(c0 + t) * d_m + d]), a);
                acc[k] = a;
            }
        }
        __syncthreads();
    }

    float *xo = Xp + (((size_t)b * parts + p) * Rstride + r) * d_m;
#pragma unroll
    for (int k = 0; k < MAXD; ++k) {
        const int d = tid + k * kBlock;
        if (d < d_m) xo[d] = acc[k];
    }
    if (tid == 0) {
        float *ml = ML + (((size_t)b * parts + p) * Rstride + r) * 2;
        ml[0] = m;
        ml[1] = l;
    }
}

// Log-sum-exp merge of the partials of one row, normalised: Xn[b,r,:].
__global__ void k_merge(const float *__restrict__ Xp, const float *__restrict__ ML, float *__restrict__ Xn,
                        int d_m, int R, int Rstride, int parts)
{
    const int d = blockIdx.x * kBlock + threadIdx.x;
    const int r = blockIdx.y, b = blockIdx.z;
    if (d >= d_m) return;
    float M = -INFINITY;
    for (int p = 0; p < parts; ++p) M = fmaxf(M, ML[(((size_t)b * parts + p) * Rstride + r) * 2]);
    float num = 0.f, den = 0.f;
    for (int p = 0; p < parts; ++p) {
        const size_t row = ((size_t)b * parts + p) * Rstride + r;
        const float mp = ML[row * 2], lp = ML[row * 2 + 1];
        if (lp > 0.f) {
            const float w = expf(mp - M);
            num = fmaf(w, Xp[row * d_m + d], num);
            den = fmaf(w, lp, den);
        }
    }
    Xn[((size_t)b * R + r) * d_m + d] = num / den;
}

// ---------------------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------------------
#define EL_DISPATCH_DTYPE(dt, ...)                                                   \
    switch (dt) {                                                                    \
    case EL_F32: { using T = float; __VA_ARGS__; } break;                            \
    case EL_F16: { using T = f16_t; __VA_ARGS__; } break;                            \
    default:     { using T = bf16_t; __VA_ARGS__; } break;                           \
    }

hipError_t launch_cout(const el_attn_ctx *ctx, const void *WoT, const void *bv, const void *bo, hipStream_t s)
{
    const int d_m = ctx->cfg.d_model, hd = ctx->hd;
    EL_DISPATCH_DTYPE(ctx->cfg.dtype,
        hipLaunchKernelGGL((k_cout<T>), dim3(cdiv(d_m, kBlock / 64)), dim3(kBlock), 0, s,
                           (const T *)bv, (const T *)bo, (const T *)WoT, ctx->w.c_out, hd, d_m));
    return hipGetLastError();
}

// 32 x 32 outputs per workgroup where that still leaves two workgroups per compute unit of a full chip, 32 x 16
// where it leaves one (less operand traffic); 16 x 16 below, where workgroups are what is missing.
// Early where all workgroups run at once and a little beyond (16 x 16 outputs: three on a compute unit; 32 x 16: two), so that nothing
// else hides the wait; straight for operands fetched four at a time and K >= 512, where a group is whole; branched for the rest.  Times of the products of 520 calls
// of d_m 256 to 1024 in proportion to the form with everything behind the length and the bias behind the last barrier, early / straight / branched:
//   16 x 16           to 512 workgroups 0.91 / 0.95 / 0.96    640 0.93 / 0.98 / 0.98    896 0.92 / 0.99 / 0.99    1024 1.04 / 0.98 / 0.98    4096 1.10 / 1.01 / 1.01
//   32 x 16, K < 512  256 0.91 / 0.96 / 0.95    512 0.95 / 0.95 / 0.94    640 1.20 / 0.96 / 0.96    K >= 512  256 0.93 / 0.88 / 0.96    512 0.93 / 0.90 / 1.03    768 1.18 / 0.94 / 1.04
//   32 x 32, K < 512  512 0.97 / 0.95 / 0.93    1024 1.04 / 0.98 / 0.98    4096 1.15 / 1.00 / 0.98       K >= 512  512 0.86 / 0.84 / 0.91    1024 0.84 / 0.82 / 0.90    4096 0.87 / 0.81 / 0.89
// (unaligned operands, 32 x 32, scores: 1.05 / 1.09 / 0.99).
template <typename TA, typename TB, typename TO>
static hipError_t launch_gemm_f32(const GemmF32 &g, int batches, hipStream_t s)
{
    auto four = [](const void *p, size_t es) { return ((uintptr_t)p & (4 * es - 1)) == 0; };
    const bool vec = g.K % 4 == 0 && g.lda % 4 == 0 && g.ldb % 4 == 0 && g.za % 4 == 0 && g.zb % 4 == 0 &&
                     four(g.A, sizeof(TA)) && four(g.Bt, sizeof(TB));
    const int tm = g.M > 16 && (long)cdiv(g.N, 16) * cdiv(g.M, 32) * batches >= 256 ? 2 : 1;
    const int tn = tm == 2 && (long)cdiv(g.N, 32) * cdiv(g.M, 32) * batches >= 512 ? 2 : 1;
    const dim3 grid(cdiv(g.N, 16 * tn), cdiv(g.M, 16 * tm), batches), block(64 * kGemmWaves);
    const bool early = (long)grid.x * grid.y * grid.z <= (tm == 1 ? 896 : 512), straight = vec && g.K >= 512;
#define EL_GEMM_F32(V, MT, NT, FORM) hipLaunchKernelGGL((k_gemm_f32<TA, TB, TO, V, MT, NT, FORM>), grid, block, 0, s, g)
#define EL_GEMM_F32_VEC(MT, NT, FORM) do { if (vec) EL_GEMM_F32(true, MT, NT, FORM); else EL_GEMM_F32(false, MT, NT, FORM); } while (0)
    if (tn == 2 && straight) EL_GEMM_F32(true, 2, 2, kGemmStraight);
    else if (tn == 2) EL_GEMM_F32_VEC(2, 2, kGemmBranched);
    else if (tm == 2 && straight) EL_GEMM_F32(true, 2, 1, kGemmStraight);
    else if (tm == 2 && early) EL_GEMM_F32_VEC(2, 1, kGemmEarly);
    else if (tm == 2) EL_GEMM_F32_VEC(2, 1, kGemmBranched);
    else if (early) EL_GEMM_F32_VEC(1, 1, kGemmEarly);
    else EL_GEMM_F32_VEC(1, 1, kGemmBranched);
#undef EL_GEMM_F32_VEC
#undef EL_GEMM_F32
    return hipGetLastError();
}

static GemmF32 gemm_args(const Problem &p, const void *A, const void *Bt, void *C, int N, int K)
{
    GemmF32 g{};
    g.A = A; g.Bt = Bt; g.C = C; g.scale = 1.0f;
    g.M = p.B * p.beam; g.N = N; g.K = K;
    g.lda = K; g.ldb = K; g.ldc = N;
    g.x = p.beam; g.R = p.R;
    g.vec_c = N % 4 == 0 && ((uintptr_t)C & 15) == 0;
    return g;
}

hipError_t launch_qproj_generic(const el_attn_ctx *ctx, const Problem &p, const Workspace &ws, hipStream_t s)
{
    GemmF32 g = gemm_args(p, p.queries, ctx->w.WqT, ws.Qp, p.hd, p.d_m);
    g.bias = ctx->w.bq;
    g.scale = 1.0f / sqrtf((float)p.d_k);
    EL_DISPATCH_DTYPE(p.dtype, return (launch_gemm_f32<T, T, float>(g, 1, s)));
    return hipErrorUnknown;
}

hipError_t launch_elq_generic(const el_attn_ctx *ctx, const Problem &p, const float *Qp, float *elq, hipStream_t s)
{
    GemmF32 g = gemm_args(p, Qp, ctx->w.Wk, elq, p.d_m, p.d_k);
    g.lda = p.hd; g.za = p.d_k; g.ldb = p.hd; g.zb = p.d_k; g.map_c = 1;
    EL_DISPATCH_DTYPE(p.dtype, return (launch_gemm_f32<float, T, float>(g, p.heads, s)));
    return hipErrorUnknown;
}

// The scores of a step take R x round_up(n, 4) floats per batch element of the region the key-range partials have
// (8 x R64 x d_m floats): with 64 rows up to n = 8 d_m, with fewer up to n = 8 d_m 64 / R.  Capacity alone decides, because
// this path is the faster one everywhere, also where one workgroup per 64 columns streams very long keys (step in us, here
// against the key-range core): one element, d_m 64, 4 rows, n 8192 93 / 140; d_m 512, 8 rows, n 8192 107 / 794, n 32768
// 364 / 3058; d_m 1024, 16 rows, n 8192 116 / 1634; d_m 30, 3 rows, n 4000 77 / 79.
bool scores_fit(const Problem &p)
{
    return (int64_t)p.R * ((p.n + 3) / 4 * 4) <= (int64_t)kMaxPartsGeneric * ((p.R + 63) / 64 * 64) * p.d_m;
}

// a3-a5 through the scores in memory; Xn normalised, one piece of statistics per row
hipError_t launch_core_scores(const el_attn_ctx *, const Problem &p, const Workspace &ws, hipStream_t s)
{
    const int64_t ldS = (p.n + 3) / 4 * 4;
    GemmF32 g = gemm_args(p, ws.ELQ, p.H, ws.Xp, p.n, p.d_m);
    g.M = p.R; g.ldc = ldS; g.za = (int64_t)p.R * p.d_m; g.zb = p.H_batch_stride; g.zc = (int64_t)p.R * ldS;
    g.lengths = p.lengths; g.use_lengths = 1; g.vec_c = 1;
    hipError_t e = hipErrorUnknown;
    EL_DISPATCH_DTYPE(p.dtype, e = (launch_gemm_f32<float, T, float>(g, p.B, s)));
    if (e != hipSuccess) return e;
    const dim3 grid(cdiv(p.d_m, 64), cdiv(p.R, 16), p.B), block(512);
    const size_t es = dtype_size(p.dtype);
    const bool vec = p.d_m % 4 == 0 && p.H_batch_stride % 4 == 0 && ((uintptr_t)p.H & (4 * es - 1)) == 0;
    EL_DISPATCH_DTYPE(p.dtype,
        if (vec) hipLaunchKernelGGL((k_sum_f32<T, true>), grid, block, 0, s, (const float *)ws.Xp, ldS, (const T *)p.H, p.H_batch_stride,
                                    p.lengths, p.n, p.d_m, p.R, ws.Xn, ws.ML);
        else hipLaunchKernelGGL((k_sum_f32<T, false>), grid, block, 0, s, (const float *)ws.Xp, ldS, (const T *)p.H, p.H_batch_stride,
                                p.lengths, p.n, p.d_m, p.R, ws.Xn, ws.ML));
    return hipGetLastError();
}

template <typename T>
static hipError_t launch_core_t(const Problem &p, const Workspace &ws, int parts, hipStream_t s)
{
    const size_t smem = (size_t)(p.d_m + kChunk) * sizeof(float);
    const dim3 grid(p.R, parts, p.B), block(kBlock);
    const float *elq = (const float *)ws.ELQ;
    const T *H = (const T *)p.H;
#define EL_CORE_CASE(MAXD)                                                                          \
    hipLaunchKernelGGL((k_core_generic<T, MAXD>), grid, block, smem, s, elq, H, p.H_batch_stride,   \
                       p.lengths, p.n, p.d_m, p.R, p.R, parts, ws.Xp, ws.ML)
    if (p.d_m <= 1 * kBlock) EL_CORE_CASE(1);
    else if (p.d_m <= 2 * kBlock) EL_CORE_CASE(2);
    else if (p.d_m <= 4 * kBlock) EL_CORE_CASE(4);
    else if (p.d_m <= 8 * kBlock) EL_CORE_CASE(8);
    else if (p.d_m <= 16 * kBlock) EL_CORE_CASE(16);
    else EL_CORE_CASE(32);
#undef EL_CORE_CASE
    return hipGetLastError();
}

hipError_t launch_core_generic(const el_attn_ctx *, const Problem &p, const Workspace &ws, int parts, hipStream_t s)
{
    EL_DISPATCH_DTYPE(p.dtype, return launch_core_t<T>(p, ws, parts, s));
    return hipErrorUnknown;
}

hipError_t launch_merge_generic(const el_attn_ctx *, const Problem &p, const Workspace &ws, int parts, int Rstride,
                                hipStream_t s)
{
    hipLaunchKernelGGL(k_merge, dim3(cdiv(p.d_m, kBlock), p.R, p.B), dim3(kBlock), 0, s,
                       (const float *)ws.Xp, (const float *)ws.ML, ws.Xn, p.d_m, p.R, Rstride, parts);
    return hipGetLastError();
}

hipError_t launch_vproj_generic(const el_attn_ctx *ctx, const Problem &p, const Workspace &ws, hipStream_t s)
{
    GemmF32 g = gemm_args(p, ws.Xn, ctx->w.WvTs, ws.A, p.d_k, p.d_m);
    g.map_a = 1; g.zb = (int64_t)p.d_k * p.d_m; g.ldc = p.hd; g.zc = p.d_k;
    EL_DISPATCH_DTYPE(p.dtype, return (launch_gemm_f32<float, T, float>(g, p.heads, s)));
    return hipErrorUnknown;
}

hipError_t launch_oproj_generic(const el_attn_ctx *ctx, const Problem &p, const Workspace &ws, const float *bias32, hipStream_t s)
{
    GemmF32 g = gemm_args(p, ws.A, ctx->w.WoTs, p.out, p.d_m, p.hd);
    g.bias32 = bias32;
    EL_DISPATCH_DTYPE(p.dtype,
        if (p.out_dtype == EL_F32) return (launch_gemm_f32<float, T, float>(g, 1, s));
        else return (launch_gemm_f32<float, T, T>(g, 1, s)));
    return hipErrorUnknown;
}

// ---------------------------------------------------------------------------------------------
// fp32 copy of a bias vector (zeros when it is absent)
template <typename T>
__global__ void k_vec_f32(const T *__restrict__ src, float *__restrict__ dst, int n)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n) dst[i] = src ? to_f32(src[i]) : 0.f;
}

hipError_t launch_vec_f32(int dtype, const void *src, float *dst, int n, hipStream_t s)
{
    EL_DISPATCH_DTYPE(dtype,
        hipLaunchKernelGGL((k_vec_f32<T>), dim3(cdiv(n, kBlock)), dim3(kBlock), 0, s, (const T *)src, dst, n));
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Segment form of the step (section 3.2: one softmax over EL-attention on a shared prefix and ordinary
// attention on each beam's own continuation).  After a1..a6 on one key set, per (query row, head):
//   seg_A   = A + b^V           the segment's own normalised head output (Eq. 8 with the probabilities
//                               summing to one inside the segment)
//   seg_lse = log sum_t exp s_t for s = Q_i K_i^T / sqrt(d_k) INCLUDING Eq. 7's key-bias term Q_i (b_i^K)^T,
//                               which is constant inside a segment (and is dropped by the step itself) but
//                               is part of the scores ordinary attention reports
// The key-range statistics (reference exponent, sum relative to it) are folded by the log-sum-exp rule
// exactly as the merge of the partials does.
// fp16 head outputs are in fragment order
template <typename T>
__device__ __forceinline__ size_t head_index(int m, int cg, int hd) { return sizeof(T) == 2 ? frag16_index(m, cg, hd) : (size_t)m * hd + cg; }

__global__ void k_seg_finish(const SegFinishArgs a)
{
    const int cg = blockIdx.x * kBlock + threadIdx.x;
    const int m = blockIdx.y;
    if (cg >= a.hd) return;
    a.seg_A[(size_t)m * a.hd + cg] = a.A[(size_t)m * a.hd + cg] + a.bv32[cg];
    if (cg % a.d_k != 0) return;
    const int i = cg / a.d_k, b = m / a.beam, j = m % a.beam, r = i * a.beam + j;
    int slot0, np;
    piece_range(a.pm, b, slot0, np);
    float M = -INFINITY;
    for (int p = 0; p < np; ++p) {
        const float *ml = a.ML + (((size_t)slot0 + p) * a.Rstride + r) * 2;
        if (ml[1] > 0.f) M = fmaxf(M, ml[0]);
    }
    float L = 0.f;
    for (int p = 0; p < np; ++p) {
        const float *ml = a.ML + (((size_t)slot0 + p) * a.Rstride + r) * 2;
        if (ml[1] > 0.f) L += expf((ml[0] - M) * a.ml_to_nat) * ml[1];
    }
    float c = 0.f;
    const float *q = a.Qp + (size_t)m * a.hd + (size_t)i * a.d_k;
    for (int k = 0; k < a.d_k; ++k) c = fmaf(q[k], a.bk32[i * a.d_k + k], c);
    a.seg_lse[(size_t)m * a.heads + i] = L > 0.f ? M * a.ml_to_nat + logf(L) + c : -INFINITY;
}

hipError_t launch_seg_finish(const SegFinishArgs &a, int rows, hipStream_t s)
{
    const dim3 grid(cdiv(a.hd, kBlock), rows), block(kBlock);
    hipLaunchKernelGGL(k_seg_finish, grid, block, 0, s, a);
    return hipGetLastError();
}

// One softmax over the union of the segments' keys, per (row, head):
//   w_s = exp(lse_s - max_s' lse_s') / sum_s' exp(lse_s' - max),   A = sum_s w_s seg_A_s      (then a7 on A)
// Bound: memory latency, one round trip for the statistics and the outputs of all segments.
template <typename TO>
__global__ void k_seg_merge(const SegMergeArgs a)
{
    const int cg = blockIdx.x * kBlock + threadIdx.x;
    const int m = blockIdx.y;
    if (cg >= a.hd) return;
    const int i = cg / a.d_k;
    float ls[kMaxSegments], x[kMaxSegments], M = -INFINITY;
    // (all requested before any is waited for)
#pragma unroll
    for (int s = 0; s < kMaxSegments; ++s) {
        ls[s] = -INFINITY; x[s] = 0.f;
        if (s < a.nseg) { ls[s] = a.lse[s][(size_t)m * a.heads + i]; x[s] = a.A[s][(size_t)m * a.hd + cg]; }
    }
#pragma unroll
    for (int s = 0; s < kMaxSegments; ++s) M = fmaxf(M, ls[s]);
    float num = 0.f, den = 0.f;
#pragma unroll
    for (int s = 0; s < kMaxSegments; ++s) {
        if (s < a.nseg && ls[s] > -INFINITY) {
            const float w = expf(ls[s] - M);
            num = fmaf(w, x[s], num);
            den += w;
        }
    }
    from_f32(den > 0.f ? num / den : 0.f, (TO *)a.A_out + head_index<TO>(m, cg, a.hd));
}

hipError_t launch_seg_merge(const SegMergeArgs &a, bool out_f16, int rows, hipStream_t s)
{
    const dim3 grid(cdiv(a.hd, kBlock), rows), block(kBlock);
    if (out_f16) hipLaunchKernelGGL((k_seg_merge<f16_t>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_seg_merge<float>), grid, block, 0, s, a);
    return hipGetLastError();
}

} // namespace el
