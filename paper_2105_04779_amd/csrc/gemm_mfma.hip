// Small-M MFMA GEMMs for the projection steps of the EL-attention decode step (steps a1, a2, a6,
// a7 of Algorithm 3's attention routine; group 2 of Table 1 -- O(d_m^2) per query, weight-read
// bound).  All four are C[m, n] = sum_k A[m, k] * Bt[n, k] with both operands contiguous along k
// (W^Q, W^V, W^O are stored transposed at prepare time for exactly this; W^K already has that shape).
//
//   a1  Qp    = (q . W^Q + b^Q) * scale   k_gemm_slab  A = queries (storage dtype), Bt = (W^Q)^T (storage dtype)
//   a2  ELQ_i = Qp_i . (W_i^K)^T          k_elq_slab   A = Qp (fp16),               Bt = W^K in fp16     per head
//                                                      (result as a high + low pair of planes in the storage type)
//   a6  A_i   = X_i . W_i^V               k_vproj      A = merge of the pieces,     W^V in fp16 fragments per head
//   a7  out   = A . W^O + c_out           k_gemm_slab  A = A (fp16),                Bt = (W^O)^T in fp16
//
// Storage-dtype operands enter the MFMA exactly (a1 runs in the storage type).  From a2 on everything
// is fp16: bf16 weights are converted once at prepare time (exact above 2^-14, |error| <= 2^-25 below),
// and the intermediates Qp, merged X and A are rounded to fp16 once each (2^-12 relative; the
// measured end-to-end error stays several times under the 2e-3 bar).  Accumulation is fp32.
//
// k_gemm_slab: a workgroup stages 32 rows of A and 32 rows of Bt over the whole K in LDS with 1 KB
// LDS-DMA pieces (full cache lines, every byte fetched once per workgroup), then its four wavefronts
// split K.  k_vproj: weights and merged rows straight in registers, see there.
// k_elq_slab: the weight slice stays in registers, operand fragments come straight from global memory
// (a2: K = d_k is tiny).
#include "el_internal.h"

namespace el {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned int u4 __attribute__((ext_vector_type(4)));

enum { C_F32 = 0, C_F16 = 1, C_BF16 = 2 };

struct GemmArgs {
    const void *A;        // activations (see a_kind)
    const void *Bt;       // weights [N rows, K contiguous], storage dtype
    void *C;
    const void *bias;     // per output column, storage dtype, may be null
    const float *bias32;  // per output column, fp32, may be null
    float scale;          // applied to (acc + bias)
    int M, N, K;          // per batch (head)
    int lda, ldb, ldc;    // row strides in elements
    int x;                // beam: logical row m = b*x + j
    int c_rB;             // k_elq_slab: padded rows per batch element of the output (logical row m, head i -> row i * x + m % x of element m / x)
};

template <bool BF> struct Frag;
template <> struct Frag<false> {
    typedef h8 type;
    static __device__ __forceinline__ f4 mfma(h8 a, h8 b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }
};
template <> struct Frag<true> {
    typedef b8 type;
    static __device__ __forceinline__ f4 mfma(b8 a, b8 b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
};

// ---------------------------------------------------------------------------------------------
// Slab GEMM: C[M, N] = A[M, K] . Bt[N, K]^T for K = 512, 768 or 1024 (rows of 1, 1.5 or 2 KB).  One workgroup
// owns a 32 x 32 output tile.  Its 64 operand rows are fetched once, whole, into LDS (row r lands
// XOR-swizzled by row_swizzle(r % 16), see dma_piece), so global traffic is full cache lines and
// (M/32 + N/32) passes over the operands in total.  Then wavefront w multiplies k-steps
// [w K/128, (w+1) K/128) for all four 16 x 16 sub-tiles, the partial tiles are added through LDS
// and wavefront w finishes sub-tile w.
template <bool BF, int CK>
__global__ void __launch_bounds__(256)
k_gemm_slab(const GemmArgs g)
{
    typedef typename Frag<BF>::type frag_t;
    __shared__ __attribute__((aligned(1024))) char S[64 * 2048];
    const int tid = threadIdx.x, l = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = l & 15, q4 = l >> 4;
    const int m0 = blockIdx.y * 32, n0 = blockIdx.x * 32;
    const int rowb = g.K * 2;
    const unsigned s_lds = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char *)S;

    // ---- stage: wavefronts 0,1 fetch the A rows, 2,3 the Bt rows ----
    if (rowb == 1536) {
        // Rows of 1.5 KB do not split into 1 KB pieces: a wavefront's 16 rows are 24 KB of contiguous LDS, filled by
        // 24 requests; lane l of request j lands at chunk position p = 64 j + l of that block, which is row
        // r = p / 96, position q = p % 96, and must hold chunk q ^ swizzle(r) of the row.
        const char *mbase = w < 2 ? (const char *)g.A : (const char *)g.Bt;
        const int first = w < 2 ? m0 + 16 * w : n0 + 16 * (w - 2);
        const int lastv = (w < 2 ? g.M : g.N) - 1, ld = w < 2 ? g.lda : g.ldb;
#pragma unroll
        for (int j = 0; j < 24; ++j) {
            const int pz = 64 * j + l, r = pz / 96, q = pz - 96 * r;
            const unsigned voff = (unsigned)min(first + r, lastv) * (unsigned)(ld * 2) + (unsigned)((q ^ row_swizzle(r)) << 4);
            dma_piece(s_lds + 16 * w * rowb + 1024 * j, voff, mbase);
        }
    } else
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int rr = 16 * w + i;
        const char *sbase;
        if (w < 2) sbase = (const char *)g.A + (size_t)min(m0 + rr, g.M - 1) * g.lda * 2;
        else sbase = (const char *)g.Bt + (size_t)min(n0 + rr - 32, g.N - 1) * g.ldb * 2;
        const unsigned voff = (unsigned)((l ^ row_swizzle(i)) << 4);
        if (rowb == 2048) dma_row_2k(s_lds + rr * rowb, voff, sbase);
        else dma_piece(s_lds + rr * rowb, voff, sbase);
    }

    // bias of this lane's four output columns (sub-tile w), fetched while the slab is in flight
    const int mt = w >> 1, nt = w & 1;
    const int ncol = n0 + 16 * nt + 4 * q4;
    float badd[4] = {0.f, 0.f, 0.f, 0.f};
    if (ncol < g.N) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (g.bias) badd[j] = BF ? to_f32(((const bf16_t *)g.bias)[ncol + j]) : to_f32(((const f16_t *)g.bias)[ncol + j]);
            if (g.bias32) badd[j] += g.bias32[ncol + j];
        }
    }

    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();

    // ---- multiply: this wavefront's quarter of K ----
    const __attribute__((address_space(3))) char *Sl = (const __attribute__((address_space(3))) char *)S;
    const int fsw = row_swizzle(r16);
    f4 acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = f4{0.f, 0.f, 0.f, 0.f};
    const int steps = g.K / 128;
    for (int st = 0; st < steps; ++st) {
        const int chunk = (4 * (w * steps + st) + q4) ^ fsw;
        const int off = r16 * rowb + (chunk << 4);
        const frag_t a0 = __builtin_bit_cast(frag_t, *(const __attribute__((address_space(3))) u4 *)(Sl + off));
        const frag_t a1 = __builtin_bit_cast(frag_t, *(const __attribute__((address_space(3))) u4 *)(Sl + off + 16 * rowb));
        const frag_t b0 = __builtin_bit_cast(frag_t, *(const __attribute__((address_space(3))) u4 *)(Sl + off + 32 * rowb));
        const frag_t b1 = __builtin_bit_cast(frag_t, *(const __attribute__((address_space(3))) u4 *)(Sl + off + 48 * rowb));
        // weights as the MFMA's A operand: the result is the transposed tile, so a lane holds four
        // consecutive output columns of one row
        acc[0][0] = Frag<BF>::mfma(b0, a0, acc[0][0]);
        acc[0][1] = Frag<BF>::mfma(b1, a0, acc[0][1]);
        acc[1][0] = Frag<BF>::mfma(b0, a1, acc[1][0]);
        acc[1][1] = Frag<BF>::mfma(b1, a1, acc[1][1]);
    }

    // ---- add the four K quarters: wavefront w collects sub-tile (mt, nt) ----
    __syncthreads();                                   // the slab is no longer needed
    float *red = (float *)S;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) *(f4 *)(red + (((w * 4) + a * 2 + b) * 64 + l) * 4) = acc[a][b];
    __syncthreads();
    f4 sum = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const f4 o = *(const f4 *)(red + (((s * 4) + mt * 2 + nt) * 64 + l) * 4);
        sum[0] += o[0]; sum[1] += o[1]; sum[2] += o[2]; sum[3] += o[3];
    }
    const int mm = m0 + 16 * mt + r16;
    if (mm >= g.M || ncol >= g.N) return;
    float val[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) val[j] = (sum[j] + badd[j]) * g.scale;
    const size_t ci = (size_t)mm * g.ldc + ncol;
    if (CK == C_F32) {
        *(f4 *)((float *)g.C + ci) = f4{val[0], val[1], val[2], val[3]};
    } else if (CK == C_F16) {
        typedef _Float16 h4 __attribute__((ext_vector_type(4)));
        *(h4 *)((f16_t *)g.C + ci) = h4{(_Float16)val[0], (_Float16)val[1], (_Float16)val[2], (_Float16)val[3]};
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) from_f32(val[j], (bf16_t *)g.C + ci + j);
    }
}

// ---------------------------------------------------------------------------------------------
// Merge of the pieces fused with a6 (A_i = X_i . W_i^V, Eq. 5 / Eq. 8).  A workgroup of eight wavefronts owns
// 16 NT of a head's 64 output columns for every `groups`-th tile of 16 rows; wavefront w contracts an eighth of
// d_m.  Its weights sit in registers in the order the matrix instruction wants them (packed so at prepare time:
// one load instruction = 1 contiguous KB), and so do its rows: a lane fetches the 16-byte fragments of its own row
// from every piece and merges them with the log-sum-exp weights it works out for that row,
//     X = sum_p (w_p l_p) Xhat_p / sum_p (w_p l_p),  w_p = 2^(m_p - M),
// so nothing is exchanged before the products are: no staging, one barrier.  Up to four pieces are in flight at a
// time; more are folded in with a running maximum.
// Bound: memory latency in a chain of two (piece table, then statistics and pieces together), then the pieces'
// bytes.  One column block per workgroup (NT = 1) where a head's four leave compute units idle: the pieces are then
// read four times, out of L2.  Against the kernel it replaces (weights and merged rows staged in LDS, one workgroup
// per 16 rows, the 128 KB of weights fetched again for every tile): 1280 rows in 448 pieces of 64 rows, d_m 1024:
// 38.9 -> 23.0 us; 512 rows, one piece each: 19.7 -> 10.2; 256 rows in 191 pieces of 64 (25 MB): 11.7 -> 10.0;
// 4 rows: 8.6 -> 5.4.
struct VprojArgs {
    const u4 *Wp;          // (W^V) in fragments: [head][k / 32][column / 16 % 4][lane]
    const f16_t *Xp;       // normalised fp16 pieces [slot, Rs, d_m]
    const float *ML;       // [slot, Rs, 2]
    f16_t *A;              // [M, heads * 64]
    PieceMap pm;
    int M, x, heads, Rs, groups;
};

template <int DM, int NT>
__global__ void __launch_bounds__(512)
k_vproj(const VprojArgs a)
{
    constexpr int KS = DM / 256;                         // 32-wide slices of k per wavefront
    constexpr int PC = 4;                                // pieces in flight
    typedef float f2 __attribute__((ext_vector_type(2)));
    __shared__ f4 red[2][8 * NT * 64];
    const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r16 = l & 15, q = l >> 4;
    // Workgroup ids that differ by a multiple of 8 share an XCD and its L2.  Heads are dealt out so that an XCD
    // works on as few of them as possible (heads / 8 when that divides): it then pulls only those heads' weights
    // from memory, once, instead of every XCD pulling all of W^V.
    constexpr int NB = 4 / NT;                           // column blocks of a head
    int head, nb, group;
    {
        const int xcd = blockIdx.x & 7, hp = (a.heads + 7) >> 3;
        int j = blockIdx.x >> 3;
        head = xcd * hp + j % hp; j /= hp;
        nb = j % NB; group = j / NB;
        if (head >= a.heads) return;
    }
    int e_tot = 0;
    if (a.pm.E) e_tot = a.pm.E[a.pm.B];
    const int tiles = (a.M + 15) >> 4;
    auto row_of = [&](int tile, int &b, int &j) { const int m = min(16 * tile + r16, a.M - 1); b = m / a.x; j = m - b * a.x; };
    int b, j, E_b = 0, E_b1 = 0;
    row_of(group, b, j);
    if (a.pm.E) { E_b = a.pm.E[b]; E_b1 = a.pm.E[b + 1]; }
    u4 wv[KS][NT];
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int t = 0; t < NT; ++t)
            wv[s][t] = a.Wp[(((size_t)head * (DM / 32) + KS * w + s) * 4 + nb * NT + t) * 64 + l];
    const PieceCut cut = piece_cut(a.pm, e_tot);
    int parity = 0;
    for (int tile = group; tile < tiles; tile += a.groups) {
        int slot0, np;
        piece_range(a.pm, cut, b, E_b, E_b1, slot0, np);
        const size_t row0 = (size_t)slot0 * a.Rs + head * a.x + j;
        int np_max = np;                                 // most pieces among the 16 rows (uniform)
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) np_max = max(np_max, __shfl_xor(np_max, o, 64));
        np_max = __builtin_amdgcn_readfirstlane(np_max);
        float v[KS][8], m_run = -INFINITY, den = 0.f;
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int e = 0; e < 8; ++e) v[s][e] = 0.f;
        for (int p0 = 0; p0 < np_max; p0 += PC) {
            f2 ml[PC];
            h8 xv[PC][KS];
#pragma unroll
            for (int p = 0; p < PC; ++p) {
                if (p0 + p >= np_max) { ml[p] = f2{0.f, 0.f}; continue; }           // uniform
                const size_t row = row0 + (size_t)min(p0 + p, np - 1) * a.Rs;
                ml[p] = *(const f2 *)(a.ML + row * 2);
#pragma unroll
                for (int s = 0; s < KS; ++s) xv[p][s] = *(const h8 *)(a.Xp + row * DM + 32 * (KS * w + s) + 8 * q);
            }
            if (p0 + PC >= np_max && tile + a.groups < tiles) {                     // the next tile's table entries
                row_of(tile + a.groups, b, j);
                if (a.pm.E) { E_b = a.pm.E[b]; E_b1 = a.pm.E[b + 1]; }
            }
            float m_new = m_run;
#pragma unroll
            for (int p = 0; p < PC; ++p) {
                if (p0 + p >= np || !(ml[p][1] > 0.f)) ml[p] = f2{-INFINITY, 0.f};  // no such piece for this row, or an empty one
                m_new = fmaxf(m_new, ml[p][0]);
            }
            if (p0 > 0) {
                const float c = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - m_new);
                den *= c;
#pragma unroll
                for (int s = 0; s < KS; ++s)
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[s][e] *= c;
            }
            m_run = m_new;
#pragma unroll
            for (int p = 0; p < PC; ++p) {
                if (p0 + p >= np_max) continue;
                const bool there = ml[p][1] > 0.f;       // an empty piece's row was never written
                const float wp = there ? exp2f(ml[p][0] - m_new) * ml[p][1] : 0.f;
                den += wp;
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    const h8 xs = there ? xv[p][s] : h8{};
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[s][e] = fmaf(wp, (float)xs[e], v[s][e]);
                }
            }
        }
        const float inv = den > 0.f ? 1.0f / den : 0.f;
        f4 acc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            h8 xm;
#pragma unroll
            for (int e = 0; e < 8; ++e) xm[e] = (_Float16)(v[s][e] * inv);
#pragma unroll
            for (int t = 0; t < NT; ++t)                 // transposed tile: lane = row, 4 columns
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, wv[s][t]), xm, acc[t], 0, 0, 0);
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) red[parity][(w * NT + t) * 64 + l] = acc[t];
        __syncthreads();                                 // the other buffer was read before this barrier's predecessor
        if (w < NT) {
            f4 sum = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < 8; ++s) sum += red[parity][(s * NT + w) * 64 + l];
            const int mm = 16 * tile + r16;
            typedef _Float16 h4 __attribute__((ext_vector_type(4)));
            if (mm < a.M)
                *(h4 *)(a.A + (size_t)mm * (a.heads * 64) + head * 64 + 16 * (nb * NT + w) + 4 * q) =
                    h4{(_Float16)sum[0], (_Float16)sum[1], (_Float16)sum[2], (_Float16)sum[3]};
        }
        parity ^= 1;
    }
}

// W^V [d_m, heads * 64] in the storage type -> fp16 fragments of k_vproj (prepare time).
template <typename T>
__global__ void k_pack_wv(const T *__restrict__ W, f16_t *__restrict__ Wp, int d_m, int hd)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (size_t)d_m * hd) return;
    const int e = i & 7, l = (i >> 3) & 63, t = (i >> 9) & 3;
    const int ks = (int)((i >> 11) % (d_m / 32)), head = (int)((i >> 11) / (d_m / 32));
    const int col = head * 64 + 16 * t + (l & 15), k = 32 * ks + 8 * (l >> 4) + e;
    Wp[i] = (f16_t)to_f32(W[(size_t)k * hd + col]);
}

hipError_t launch_pack_wv(int dtype, const void *W, void *Wp, int d_m, int hd, hipStream_t s)
{
    const dim3 grid((unsigned)(((size_t)d_m * hd + 255) / 256)), block(256);
    if (dtype == EL_BF16) hipLaunchKernelGGL(k_pack_wv<bf16_t>, grid, block, 0, s, (const bf16_t *)W, (f16_t *)Wp, d_m, hd);
    else hipLaunchKernelGGL(k_pack_wv<f16_t>, grid, block, 0, s, (const f16_t *)W, (f16_t *)Wp, d_m, hd);
    return hipGetLastError();
}

// bf16 -> fp16 copy of a weight matrix (prepare time).
__global__ void k_bf16_to_f16(const bf16_t *src, f16_t *dst, size_t n)   // src may equal dst
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) dst[i] = (f16_t)to_f32(src[i]);
}

hipError_t launch_bf16_to_f16(const void *src, void *dst, size_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_bf16_to_f16, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, (const bf16_t *)src, (f16_t *)dst, n);
    return hipGetLastError();
}

// Transpose a [rows, cols] matrix of 16- or 32-bit elements (prepare-time packing of W^Q, W^V, W^O).
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
// ---------------------------------------------------------------------------------------------
// a2, query expansion (Eq. 9's Q_i (W_i^K)^T): ELQ[b, i*x + j, :] = Qp[b*x + j, head i] . (W_i^K)^T with
// d_k = 64.  One workgroup owns 64 output columns of one head for up to 256 logical rows: its slice
// of W^K (64 x 64, 8 KB) is read once and stays in registers as MFMA fragments while the four
// wavefronts walk over the row tiles, so W^K is read once per 256 rows instead of once per 16.
// Weights are the MFMA's A operand: a lane ends up with four consecutive columns of one row; the
// 16 x 64 tile then goes through LDS and leaves in the fragment order of the attention core (elq_frag_index),
// 64 contiguous bytes per row and 32-column fragment.
template <bool BF>
__global__ void __launch_bounds__(256)
k_elq_slab(const GemmArgs g)
{
    typedef uint16_t q4 __attribute__((ext_vector_type(4)));
    constexpr int MT = 4;                               // row tiles per wavefront
    __shared__ __attribute__((aligned(16))) uint16_t Ct[2][4][MT][16 * 72];   // [plane]; rows 144 bytes apart

    const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int r16 = l & 15, qd = l >> 4;
    const int n0 = blockIdx.x * 64, head = blockIdx.y;
    const int mt0 = blockIdx.z * (4 * MT);              // first 16-row tile of this workgroup

    u4 bfr[4][2], afr[MT][2];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int u = 0; u < 2; ++u)
            bfr[t][u] = *(const u4 *)((const f16_t *)g.Bt + (size_t)(n0 + 16 * t + r16) * g.ldb + head * 64 + 32 * u + 8 * qd);
#pragma unroll
    for (int mi = 0; mi < MT; ++mi) {
        const int m = min((mt0 + w + 4 * mi) * 16 + r16, g.M - 1);
#pragma unroll
        for (int u = 0; u < 2; ++u)
            afr[mi][u] = *(const u4 *)((const f16_t *)g.A + (size_t)m * g.lda + head * 64 + 32 * u + 8 * qd);
    }
#pragma unroll
    for (int mi = 0; mi < MT; ++mi) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int u = 0; u < 2; ++u)
                acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, bfr[t][u]), __builtin_bit_cast(h8, afr[mi][u]), acc, 0, 0, 0);
            q4 hi, lo;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                uint16_t h, l2;
                split16<BF>(acc[e], h, l2);
                hi[e] = h; lo[e] = l2;
            }
            *(q4 *)(&Ct[0][w][mi][r16 * 72 + 16 * t + 4 * qd]) = hi;
            *(q4 *)(&Ct[1][w][mi][r16 * 72 + 16 * t + 4 * qd]) = lo;
        }
    }
    // a wavefront reads back only what it wrote: no barrier.  Eight lanes write one 128-byte row piece.
#pragma unroll
    for (int mi = 0; mi < MT; ++mi) {
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
            const int row = 8 * hf + (l >> 3), m = (mt0 + w + 4 * mi) * 16 + row;
            if (m >= g.M) continue;
            uint16_t *dst = (uint16_t *)g.C + elq_frag_index(m / g.x, head * g.x + m % g.x, n0 + 8 * (l & 7), 0, g.c_rB, g.ldc);
            *(u4 *)dst = *(const u4 *)(&Ct[0][w][mi][row * 72 + 8 * (l & 7)]);
            *(u4 *)(dst + 512) = *(const u4 *)(&Ct[1][w][mi][row * 72 + 8 * (l & 7)]);
        }
    }
}

bool gemm_mfma_supported(int dtype, int d_m, int d_k)
{
    return (dtype == EL_F16 || dtype == EL_BF16) && (d_m == 512 || d_m == 768 || d_m == 1024) && d_k == 64;
}

static GemmArgs base_args(const Problem &p)
{
    GemmArgs g{};
    g.scale = 1.0f;
    g.x = p.beam;
    g.M = p.B * p.beam;
    return g;
}

template <bool BF, int CK>
static hipError_t launch_slab(const GemmArgs &g, hipStream_t s)
{
    hipLaunchKernelGGL((k_gemm_slab<BF, CK>), dim3((g.N + 31) / 32, (g.M + 31) / 32), dim3(256), 0, s, g);
    return hipGetLastError();
}

// a1: Qp = (q . W^Q + b^Q) * scale        [B*beam, hd] fp16
hipError_t launch_qproj_mfma(const el_attn_ctx *ctx, const Problem &p, const Workspace &ws, float scale, hipStream_t s)
{
    GemmArgs g = base_args(p);
    g.A = p.queries; g.Bt = ctx->w.WqT; g.C = ws.Qp; g.bias = ctx->w.bq; g.scale = scale;
    g.N = p.hd; g.K = p.d_m; g.lda = p.d_m; g.ldb = p.d_m; g.ldc = p.hd;
    return p.dtype == EL_BF16 ? launch_slab<true, C_F16>(g, s) : launch_slab<false, C_F16>(g, s);
}

// a2: ELQ[b, i*beam+j, :] = Qp[b*beam+j, head i] . (W_i^K)^T      high + low planes in fragment order, Rs rows per b
hipError_t launch_elq_mfma(const el_attn_ctx *ctx, const Problem &p, const Workspace &ws, int Rs, hipStream_t s)
{
    GemmArgs g = base_args(p);
    g.A = ws.Qp; g.Bt = ctx->w.WkH; g.C = ws.ELQ;
    g.N = p.d_m; g.K = p.d_k; g.lda = p.hd; g.ldb = p.hd; g.ldc = p.d_m;
    g.c_rB = Rs;
    const dim3 grid(p.d_m / 64, p.heads, (g.M + 255) / 256);
    if (p.dtype == EL_BF16) hipLaunchKernelGGL(k_elq_slab<true>, grid, dim3(256), 0, s, g);
    else hipLaunchKernelGGL(k_elq_slab<false>, grid, dim3(256), 0, s, g);
    return hipGetLastError();
}

// merge + a6: A[b*beam+j, head i] = (sum_p w_p Xp[b,p,i*beam+j,:]) . W_i^V       fp16   (d_k = 64)
template <int DM>
static void launch_vproj_t(const VprojArgs &a, int nt, hipStream_t s)
{
    const dim3 grid(8 * ((a.heads + 7) / 8) * (4 / nt) * a.groups), block(512);
    if (nt == 1) hipLaunchKernelGGL((k_vproj<DM, 1>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_vproj<DM, 4>), grid, block, 0, s, a);
}

hipError_t launch_vproj_mfma(const el_attn_ctx *ctx, const Problem &p, const Workspace &ws, const CorePlan &pl,
                             hipStream_t s)
{
    VprojArgs a;
    a.Wp = (const u4 *)ctx->w.WvP; a.Xp = (const f16_t *)ws.Xp; a.ML = ws.ML; a.A = (f16_t *)ws.A;
    a.pm = piece_map(pl, ws, p.B);
    a.M = p.B * p.beam; a.x = p.beam; a.heads = p.heads; a.Rs = pl.Rs;
    const int tiles = (a.M + 15) / 16;
    const int nt = tiles * p.heads <= 64 ? 1 : 4;
    const int room = ctx->num_cus / p.heads > 0 ? ctx->num_cus / p.heads : 1;
    a.groups = tiles < room ? tiles : room;
    if (p.d_m == 1024) launch_vproj_t<1024>(a, nt, s);
    else if (p.d_m == 768) launch_vproj_t<768>(a, nt, s);
    else launch_vproj_t<512>(a, nt, s);
    return hipGetLastError();
}

// a7: out = A . W^O + c_out
hipError_t launch_oproj_mfma(const el_attn_ctx *ctx, const Problem &p, const Workspace &ws, const float *bias32, hipStream_t s)
{
    GemmArgs g = base_args(p);
    g.A = ws.A; g.Bt = ctx->w.WoT; g.C = p.out; g.bias32 = bias32;
    g.N = p.d_m; g.K = p.hd; g.lda = p.hd; g.ldb = p.hd; g.ldc = p.d_m;
    if (p.out_dtype == EL_F32) return launch_slab<false, C_F32>(g, s);
    if (p.dtype == EL_BF16) return launch_slab<false, C_BF16>(g, s);
    return launch_slab<false, C_F16>(g, s);
}

} // namespace el
