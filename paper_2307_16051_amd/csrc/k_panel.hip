// k_panel.hip -- the no-interchange factorisation of one outer block (up to
// 1024 columns) for FP16 / BF16 storage: Gaussian elimination (Section 1.3)
// on the half-precision copy of the Jacobian (Section 2), checked on the fly
// against partial pivoting as in k_getrf.hip (every Schur-complement entry
// below a pivot must satisfy |a_ik| <= (1 - 2^-8) |a_kk|, i.e. every
// multiplier |l_ik| <= 1 - 2^-8; a failure sets FLAG_FAIL and the host
// factors again with explicit pivoting).
//
// For the outer block with columns [k0, k0 + W):
//   k_top   factors its W x W diagonal square A11 = L11 U11.  One workgroup
//           per 64-row tile, holding the tile's W columns in LDS.  Leaf l
//           (columns 64 l .. 64 l + 63) is factored by workgroup l, which
//           also inverts its triangular factors and forms the leaf's U row
//           block; the workgroups below take their L tile X U^{-1} and their
//           rank-64 update from what it publishes.  Everything a leaf passes
//           on travels as 64-bit words stamped with the leaf's tag (no flag
//           round trip, no cache-wide fence).
//   k_trsm  L21 = A21 U11^{-1} for the 64-row tiles below the square
//           (left-looking over the leaves) and U12 = L11^{-1} A12 for the
//           64-column slabs to its right (block forward substitution).
// The trailing update A22 -= L21 U12 (K = W) is the matrix-core GEMM of
// k_getrf.hip.
//
// Products run on the matrix cores (v_mfma_f32_32x32x16_{f16,bf16}, FP32
// accumulation).  A product with a triangular inverse splits the FP32 inverse
// (scaled by a power of two) into a high and a low half-precision part, and
// an FP32 right-hand side likewise, so it carries about 16-22 bits before the
// result is rounded once to the storage type -- the accuracy of the FP32
// substitution it replaces, not that of half precision.
#include <algorithm>

#include "n3p_gemm.hpp"

namespace n3p {

namespace {

constexpr int PT = 64;               // leaf width and tile height
constexpr int TOP_THREADS = 512;     // eight wavefronts
constexpr int TRSM_THREADS = 512;    // eight wavefronts
constexpr int PSPIN = 1 << 22;       // bounded polls (~0.1 s): a wait that long has failed

// publication words of one leaf (64-bit: tag << 32 | two storage values).
// A 64x64 block published as a matrix-core operand (rows m, depth k) takes
// 2048 words: the pair (k, k + 1) of row m = 32 fm + l32 with
// k = 16 ks + 8 h + 2 e is word op_word(fm, ks, h, l32, e), so the four words
// a lane reads per 16-deep step are adjacent and a wavefront's read of one
// step is 2 KB contiguous.
constexpr int PUB_UINV = 0;          // (U^{-1} * 2^s)^T: high parts, then low parts at + 2048
constexpr int PUB_SCALE = 4096;      // s (four copies)
constexpr int PUB_U12 = 4160;        // + 2048 b: U(leaf, b)^T, the leaf's U rows in block column b
constexpr int PUB_LEAF = PUB_U12 + 16 * 2048;
__host__ __device__ constexpr int op_word(int fm, int ks, int h, int l32, int e)
{
    return (((fm * 4 + ks) * 2 + h) * 32 + l32) * 4 + e;
}
// side buffer for k_trsm (storage type): per leaf the scaled high and low
// parts of (U^{-1})^T and of L^{-1} as matrix-core operands (the pair of word
// op_word(...) at elements 2 op_word(...), + 1); after the 16 leaves, two int
// exponents per leaf (s of U^{-1}, s of L^{-1})
constexpr int IH_UHI = 0, IH_ULO = 4096, IH_LHI = 8192, IH_LLO = 12288, IH_LEAF = 16384;
constexpr int IH_EXP = 16 * IH_LEAF;  // element offset of the exponents (as int pairs)
// then copies of the square's off-diagonal blocks in matrix-core operand
// order, for k_trsm: block (r, b) at OP_U + (16 r + b) * 4096 holds U(r, b)^T
// (b > r) and at OP_L + (16 r + b) * 4096 L(r, b) (b < r); element p of
// lane (h, l32) of 16-deep step ks of row half fm is at
// ((4 fm + ks) * 64 + 32 h + l32) * 8 + p, so one wavefront's operand load
// is 1 KB contiguous
constexpr int OP_U = IH_EXP + 128;
constexpr int OP_L = OP_U + 256 * 4096;
constexpr int IH_TOTAL = OP_L + 256 * 4096;

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// 32x32x16 matrix-core step.  Operands: lane l holds row (A) / column (B)
// l & 31 and the 8 consecutive K values 8 (l >> 5) .. +7 of the 16-deep step;
// result: lane l holds column l & 31, rows 8 g + 4 (l >> 5) + q in acc[4 g + q].
template <typename T> struct pmma;
template <> struct pmma<f16> {
    typedef h8 vec;
    static __device__ __forceinline__ f32x16 op(vec a, vec b, f32x16 c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
    }
};
template <> struct pmma<bf16> {
    typedef b8 vec;
    static __device__ __forceinline__ f32x16 op(vec a, vec b, f32x16 c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
};

template <typename T> __device__ __forceinline__ uint32_t bits(T v)
{
    return (uint32_t)__builtin_bit_cast(unsigned short, v);
}
template <typename T> __device__ __forceinline__ T from_bits(uint32_t b)
{
    return __builtin_bit_cast(T, (unsigned short)(b & 0xffffu));
}
template <typename T> __device__ __forceinline__ uint32_t pack2(T a, T b)
{
    return bits(a) | (bits(b) << 16);
}
template <typename T> __device__ __forceinline__ typename pmma<T>::vec as_vec(u32x4 v)
{
    return __builtin_bit_cast(typename pmma<T>::vec, v);
}
// 1/v: hardware reciprocal estimate refined by one Newton-Raphson step (within
// an ulp of the rounded quotient; the pivots of the leaf chain)
__device__ __forceinline__ float rcp_nr(float v)
{
    const float r = __builtin_amdgcn_rcpf(v);
    return fmaf(fmaf(-v, r, 1.0f), r, r);
}
__device__ __forceinline__ f32x16 zero16()
{
    f32x16 z;
#pragma unroll
    for (int q = 0; q < 16; ++q) z[q] = 0.0f;
    return z;
}

// high / low storage-precision parts of 8 FP32 values (v ~ hi + lo)
template <typename T>
__device__ __forceinline__ void split8(const float (&v)[8], typename pmma<T>::vec &hi,
                                       typename pmma<T>::vec &lo)
{
    u32x4 a, b;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const T h0 = (T)v[2 * p], h1 = (T)v[2 * p + 1];
        const T l0 = (T)(v[2 * p] - to_f32(h0)), l1 = (T)(v[2 * p + 1] - to_f32(h1));
        a[p] = pack2(h0, h1);
        b[p] = pack2(l0, l1);
    }
    hi = as_vec<T>(a);
    lo = as_vec<T>(b);
}

// power-of-two exponent s with max * 2^s in [2^13, 2^14) (0 for a zero max)
__device__ __forceinline__ int scale_exp(float mx)
{
    if (!(mx > 0.0f) || !isfinite(mx)) return 0;
    int e;
    frexpf(mx, &e);
    return 14 - e;
}

// Element (i, c) of a tile with rows of W values held row-major in LDS.  The
// 16-byte chunks of row i are permuted by XOR with i & 7, so 8 consecutive
// rows of one column, and one column chunk of 32 consecutive rows, spread
// over the banks.  Chunks stay 16-byte aligned.
__device__ __forceinline__ int tix(int i, int c, int W)
{
    return i * W + ((((c >> 3) ^ (i & 7)) << 3) | (c & 7));
}

__device__ __forceinline__ uint64_t tload(const uint64_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void tstore(uint64_t *p, uint32_t tag, uint32_t v)
{
    __hip_atomic_store(p, ((uint64_t)tag << 32) | v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// NG groups of 4 consecutive words per lane (group g at base + g * stride):
// poll until every word of the wavefront carries `tag` (bounded; an expired
// wait raises FLAG_TIMEOUT and returns whatever was read).
template <int NG>
__device__ __forceinline__ void tissue4(const uint64_t *base, int stride, uint64_t (&v)[NG][4])
{
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e) v[g][e] = tload(base + g * stride + e);
}
// the wait of tfetch4 on words already issued by tissue4
template <int NG>
__device__ __forceinline__ void twait4(uint64_t (&v)[NG][4], const uint64_t *base, int stride,
                                       uint32_t tag, uint32_t (&out)[NG][4], int *flags)
{
    int spins = 0;
    for (;;) {
        bool ok = true;
#pragma unroll
        for (int g = 0; g < NG; ++g)
#pragma unroll
            for (int e = 0; e < 4; ++e) ok &= (uint32_t)(v[g][e] >> 32) == tag;
        if (__all(ok)) break;
        if (++spins > PSPIN) {
            set_flag(&flags[FLAG_TIMEOUT], 1);
            break;
        }
        __builtin_amdgcn_s_sleep(1);
#pragma unroll
        for (int g = 0; g < NG; ++g)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if ((uint32_t)(v[g][e] >> 32) != tag) v[g][e] = tload(base + g * stride + e);
    }
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e) out[g][e] = (uint32_t)v[g][e];
}
template <int NG>
__device__ __forceinline__ void tfetch4(const uint64_t *base, int stride, uint32_t tag,
                                        uint32_t (&out)[NG][4], int *flags)
{
    uint64_t v[NG][4];
    tissue4<NG>(base, stride, v);
    twait4<NG>(v, base, stride, tag, out, flags);
}

template <typename T> __device__ __forceinline__ u32x4 to_u4(const uint32_t (&w)[4])
{
    u32x4 v;
    v[0] = w[0];
    v[1] = w[1];
    v[2] = w[2];
    v[3] = w[3];
    return v;
}

// Max over a wavefront (every lane active) with DPP row operations: two quad
// swaps, then the half-row and row mirrors leave each 16-lane row's max in
// all of its lanes; the four rows are combined through lane reads.  (Max is
// exact, so the order of the comparisons does not change the result.)
__device__ __forceinline__ float dpp_f(float v, int ctrl_sel)
{
    const int b = __float_as_int(v);
    int r;
    switch (ctrl_sel) {
    case 0: r = __builtin_amdgcn_update_dpp(b, b, 0xB1, 0xF, 0xF, false); break;   // quad_perm [1,0,3,2]
    case 1: r = __builtin_amdgcn_update_dpp(b, b, 0x4E, 0xF, 0xF, false); break;   // quad_perm [2,3,0,1]
    case 2: r = __builtin_amdgcn_update_dpp(b, b, 0x141, 0xF, 0xF, false); break;  // row_half_mirror
    default: r = __builtin_amdgcn_update_dpp(b, b, 0x140, 0xF, 0xF, false); break; // row_mirror
    }
    return __int_as_float(r);
}
__device__ __forceinline__ float wave_max(float v)
{
    v = fmaxf(v, dpp_f(v, 0));
    v = fmaxf(v, dpp_f(v, 1));
    v = fmaxf(v, dpp_f(v, 2));
    v = fmaxf(v, dpp_f(v, 3));
    const float a = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0));
    const float b = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 16));
    const float c = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 32));
    const float d = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 48));
    return fmaxf(fmaxf(a, b), fmaxf(c, d));
}

typedef float DmRow[PT + 1];

// Triangular inverses in place in Dm: U^{-1} on and above the diagonal,
// L^{-1} (unit diagonal, not stored) below it.  Waves 0..3 take U, waves
// 4..7 L: the four diagonal 16x16 blocks by substitution, one per wave, then
// 16 -> 32 -> 64: for a pair of inverted diagonal blocks X11, X22 and the
// block U12 (L21) between them, X12 = -X11 (U12 X22), X21 = -X22 (L21 X11)
// on v_mfma_f32_16x16x4f32, the inner product staying in the registers it was
// formed in.  This is on the chain of leaves: 3.4 us a leaf with the scale
// exponents, 6.0 us with 8x8 blocks, a doubling on the VALU, two that passed
// the inner products through LDS and a scan for the exponents.  Each step
// returns the largest magnitude this lane wrote.

// Element (i, m) of the triangle's inverse, its zeros and unit diagonal filled in.
__device__ __forceinline__ float tri_at(const DmRow *Dm, int tri, int i, int m)
{
    const float x = Dm[i][m];
    return tri == 0 ? (m >= i ? x : 0.0f) : (m < i ? x : (m == i ? 1.0f : 0.0f));
}

// The 16x16 diagonal blocks, by substitution: wave 4 tri + q block q.  The
// four lanes 4 c + g of a quad share column c: lane g keeps the entries of
// rows 4 j + g and sums their part of each row's product, and the quad adds
// up (with one lane per column, a quarter of the lanes, the 120 products and
// their operands took 2 us).  A wave reads and writes its own triangle only.
__device__ __forceinline__ float inv_diag16(DmRow *Dm, int w, int lane)
{
    const int b = 16 * (w & 3), c = lane >> 2, g = lane & 3;
    float xg[4] = {0.0f, 0.0f, 0.0f, 0.0f}, mx = 0.0f;
    auto quad_sum = [](float v) {
        v += dpp_f(v, 0);
        return v + dpp_f(v, 1);
    };
    if (w < 4) {
        float rd[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) rd[j] = rcp_nr(Dm[b + 4 * j + g][b + 4 * j + g]);
#pragma unroll
        for (int r = 15; r >= 0; --r) {
            const int j0 = r >> 2;
            float s = 0.0f;
#pragma unroll
            for (int j = 3; j > j0; --j) s += Dm[b + r][b + 4 * j + g] * xg[j];
            const float ub = Dm[b + r][b + 4 * j0 + g];
            s += (g > (r & 3) ? ub : 0.0f) * xg[j0];
            float rr;
            switch (r & 3) {
            case 0: rr = quad_bcast<0>(rd[j0]); break;
            case 1: rr = quad_bcast<1>(rd[j0]); break;
            case 2: rr = quad_bcast<2>(rd[j0]); break;
            default: rr = quad_bcast<3>(rd[j0]); break;
            }
            const float x = ((r == c ? 1.0f : 0.0f) - quad_sum(s)) * rr;
            xg[j0] = g == (r & 3) ? x : xg[j0];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (4 * j + g <= c) {
                Dm[b + 4 * j + g][b + c] = xg[j];
                mx = fmaxf(mx, fabsf(xg[j]));
            }
    } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int j0 = r >> 2;
            float s = 0.0f;
#pragma unroll
            for (int j = 0; j < j0; ++j) s += Dm[b + r][b + 4 * j + g] * xg[j];
            const float lb = Dm[b + r][b + 4 * j0 + g];
            s += (g < (r & 3) ? lb : 0.0f) * xg[j0];
            const float x = (r == c ? 1.0f : 0.0f) - quad_sum(s);
            xg[j0] = g == (r & 3) ? x : xg[j0];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (4 * j + g > c) {
                Dm[b + 4 * j + g][b + c] = xg[j];
                mx = fmaxf(mx, fabsf(xg[j]));
            }
    }
    return mx;
}

// 16x16 tile of A B (K = k_len, a multiple of 4) on the FP32 matrix cores
// (v_mfma_f32_16x16x4f32): lane l supplies A[l & 15][k + (l >> 4)] and
// B[k + (l >> 4)][l & 15] for each 4-deep step; the result acc[q] is the entry
// (4 (l >> 4) + q, l & 15).
template <int KL, typename FA, typename FB>
__device__ __forceinline__ f32x4 mm16f32(FA fa, FB fb, int lane)
{
    f32x4 acc;
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] = 0.0f;
    const int ci = lane & 15, kq = lane >> 4;
    // every operand read first, then the products in order
    float av[KL / 4], bv[KL / 4];
#pragma unroll
    for (int s = 0; s < KL / 4; ++s) {
        av[s] = fa(ci, 4 * s + kq);
        bv[s] = fb(4 * s + kq, ci);
    }
#pragma unroll
    for (int s = 0; s < KL / 4; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[s], bv[s], acc, 0, 0, 0);
    return acc;
}

// acc - P T, T a 16x16 fragment as mm16f32 left it: register q of lane l
// holds row 4 (l >> 4) + q of T, so step q takes that column of P
template <typename FP>
__device__ __forceinline__ f32x4 mm16_sub(f32x4 acc, FP fp, const f32x4 &t, int lane)
{
    const int ci = lane & 15, kq = lane >> 4;
    float pv[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) pv[q] = -fp(ci, 4 * kq + q);
#pragma unroll
    for (int q = 0; q < 4; ++q) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(pv[q], t[q], acc, 0, 0, 0);
    return acc;
}
// Doubling BS -> 2 BS.  BS = 16: waves 0, 1 (U) and 4, 5 (L), one pair of
// blocks each.  BS = 32: wave 4 tri + 2 ti + tc the 16x16 tile (ti, tc); a
// barrier parts the reads of U12 (L21) from the writes in its place.
template <int BS>
__device__ __forceinline__ float inv_double(DmRow *Dm, int w, int lane)
{
    constexpr int NT = BS / 16;  // tiles per side
    const int tri = w >> 2, item = w & 3;
    const int p = BS == 16 ? 32 * item : 0, ti = BS == 16 ? 0 : item >> 1, tc = BS == 16 ? 0 : item & 1;
    // the coupling block's rows and columns, and the triangle left of the
    // inner product (rows) and inside it (columns)
    const int ra = tri == 0 ? p : p + BS, cb = tri == 0 ? p + BS : p;
    const bool on = BS == 32 || item < 2;
    f32x4 x = {0.0f, 0.0f, 0.0f, 0.0f};
    if (on) {
#pragma unroll
        for (int h = 0; h < NT; ++h) {
            if (tri == 0 ? h < ti : h > ti) continue;  // a zero tile of the left triangle
            const f32x4 t = mm16f32<BS>([&](int i, int m) { return Dm[ra + 16 * h + i][cb + m]; },
                                        [&](int m, int c) { return tri_at(Dm, tri, cb + m, cb + 16 * tc + c); },
                                        lane);
            x = mm16_sub(x, [&](int i, int m) { return tri_at(Dm, tri, ra + 16 * ti + i, ra + 16 * h + m); }, t, lane);
        }
    }
    if constexpr (BS == 32) __syncthreads();
    float mx = 0.0f;
    if (on) {
        const int ci = lane & 15, kq = lane >> 4;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            Dm[ra + 16 * ti + 4 * kq + q][cb + 16 * tc + ci] = x[q];
            mx = fmaxf(mx, fabsf(x[q]));
        }
    }
    return mx;
}

struct TopArgs {
    int64_t k0;      // first row and column of the diagonal square
    int W;           // its size (multiple of 64, <= 1024)
    void *A;         // factor matrix, column-major
    int64_t lda;
    void *LT;        // L rows, row-major, ld NB_OUT (column index relative to k0)
    uint64_t *pub;   // PUB_LEAF words per leaf
    void *inv;       // side buffer: the inverses for k_trsm
    int *flags;
    uint32_t tag0;   // leaf l publishes with tag0 + l (tags never repeat within a factorisation)
};

// ======================================================================= k_top
// LDS of the square's workgroup: the row tile, the diagonal block (FP32), a
// leaf's published U^{-1} as an operand, the waves' maxima, the check's flag
// and the exponent.
constexpr int TOP_TILE_BYTES = PT * NB_OUT * 2;
constexpr int TOP_DM_BYTES = PT * (PT + 1) * 4;
constexpr int TOP_UOP_BYTES = 2 * 6 * 64 * 16;
constexpr int TOP_LDS_BYTES = TOP_TILE_BYTES + TOP_DM_BYTES + TOP_UOP_BYTES + 32 + 16;

// Workgroup r of the diagonal square (see the file comment).  lds: at least
// TOP_LDS_BYTES, 16-byte aligned.
template <typename T>
__device__ __forceinline__ void top_body(const TopArgs &a, int r, char *lds)
{
    typedef typename pmma<T>::vec vec;
    T *tile = (T *)lds;
    DmRow *Dm = (DmRow *)(lds + TOP_TILE_BYTES);
    u32x4 *uop = (u32x4 *)(lds + TOP_TILE_BYTES + TOP_DM_BYTES);  // [high, low][six pieces][lane]
    float *red = (float *)(lds + TOP_TILE_BYTES + TOP_DM_BYTES + TOP_UOP_BYTES);
    int &sfail = *(int *)(lds + TOP_TILE_BYTES + TOP_DM_BYTES + TOP_UOP_BYTES + 32);
    int &usc = *(int *)(lds + TOP_TILE_BYTES + TOP_DM_BYTES + TOP_UOP_BYTES + 36);
    if (block_flag(&a.flags[FLAG_FAIL])) return;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, h = lane >> 5, l32 = lane & 31;
    const int W = a.W, nl = W / PT;
    T *A = (T *)a.A;
    const int64_t lda = a.lda, k0 = a.k0, row0 = k0 + (int64_t)r * PT;
    int *flags = a.flags;
    const float margin = 1.0f - 1.0f / 256.0f;

    // ---- the row tile: rows row0 .. row0 + 63, columns k0 .. k0 + W - 1
    for (int e = t; e < W * 8; e += TOP_THREADS) {
        const int c = e >> 3, rc = e & 7;
        const u32x4 v = *(const u32x4 *)(A + (row0 + rc * 8) + (k0 + c) * lda);
#pragma unroll
        for (int q = 0; q < 8; ++q) tile[tix(rc * 8 + q, c, W)] = from_bits<T>(v[q >> 1] >> (16 * (q & 1)));
    }
    if (t == 0) sfail = 0;
    __syncthreads();

    bool bad = false;
    uint64_t pre[4][4];  // words requested ahead (see below)
    // L tile of leaf l: L^T = (U^{-1})^T X^T on waves 0..3 (fm: leaf columns,
    // fn: tile rows), from the published scaled U^{-1} halves.  Every wave
    // fetches its share of the words, each word once per workgroup, and passes
    // it on through LDS: wave w the part w & 1 (high, low) of step pair
    // (w >> 1) of the three that are not zero ((fm, ks) = (0, 0..1), (1, 0..1),
    // (1, 2..3)), waves 6, 7 the exponent.  (With waves 0..3 each fetching the
    // 36 words per lane of their products, twice over, a poll of the words took
    // 1.8 us, and every workgroup below polls them.)
    auto l21 = [&](int l) {
        const uint64_t *pl = a.pub + (size_t)l * PUB_LEAF;
        const uint32_t tag = a.tag0 + (uint32_t)l;
        f32x16 acc = zero16();
        float sc = 1.0f;
        const int fm = w & 1, fn = (w >> 1) & 1, i = 32 * fn + l32;
        if (w < 6) {
            const int lo = w & 1, q = w >> 1, qf = q > 0, q0 = q == 2 ? 2 : 0;
            const uint64_t *src = pl + PUB_UINV + 2048 * lo + op_word(qf, q0, h, l32, 0);
            uint32_t v[2][4];
            tfetch4<2>(src, op_word(0, 1, 0, 0, 0), tag, v, flags);
            uop[(lo * 6 + 2 * q) * 64 + lane] = to_u4<T>(v[0]);
            uop[(lo * 6 + 2 * q + 1) * 64 + lane] = to_u4<T>(v[1]);
        } else if (w == 6) {
            uint32_t se[1][4];
            tfetch4<1>(pl + PUB_SCALE, 0, tag, se, flags);
            if (lane == 0) usc = (int)se[0][0];
        }
        __syncthreads();
        if (w < 4) {
            sc = ldexpf(1.0f, -usc);
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                if (ks < 2 + 2 * fm) {  // U^{-1} is zero beyond
                    const vec b = as_vec<T>(*(const u32x4 *)&tile[tix(i, 64 * l + 16 * ks + 8 * h, W)]);
                    acc = pmma<T>::op(as_vec<T>(uop[(2 * fm + ks) * 64 + lane]), b, acc);
                    acc = pmma<T>::op(as_vec<T>(uop[(6 + 2 * fm + ks) * 64 + lane]), b, acc);
                }
            }
        }
        __syncthreads();  // every read of X done before L overwrites it
        if (w < 4) {
            bool f = false;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                T o[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float v = acc[4 * g + q] * sc;
                    f |= !(fabsf(v) <= margin);
                    o[q] = (T)v;
                }
                u32x2 st;
                st[0] = pack2(o[0], o[1]);
                st[1] = pack2(o[2], o[3]);
                *(u32x2 *)&tile[tix(i, 64 * l + 32 * fm + 8 * g + 4 * h, W)] = st;
            }
            if (f) set_flag(&flags[FLAG_FAIL], 1);
        }
        __syncthreads();
    };
    // Updates of 32 columns (half hf) of block column b, row half fn of the
    // tile: acc += U(l, b)^T L(r, l)^T for leaf l from its words, then C^T -= acc
    // (one rounding for all the leaves in acc).
    constexpr int wstr = op_word(0, 1, 0, 0, 0);
    auto u_words = [&](int l, int b, int hf) {
        return a.pub + (size_t)l * PUB_LEAF + PUB_U12 + b * 2048 + op_word(hf, 0, h, l32, 0);
    };
    auto upd_product = [&](f32x16 &acc, int l, int fn, const uint32_t (&uw)[4][4]) {
        const int i = 32 * fn + l32;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const vec lb = as_vec<T>(*(const u32x4 *)&tile[tix(i, 64 * l + 16 * ks + 8 * h, W)]);
            acc = pmma<T>::op(as_vec<T>(to_u4<T>(uw[ks])), lb, acc);
        }
    };
    auto upd_store = [&](const f32x16 &acc, int b, int hf, int fn) {
        const int i = 32 * fn + l32;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            u32x2 *p = (u32x2 *)&tile[tix(i, 64 * b + 32 * hf + 8 * g + 4 * h, W)];
            const u32x2 cv = *p;
            T o[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                o[q] = (T)(to_f32(from_bits<T>(cv[q >> 1] >> (16 * (q & 1)))) - acc[4 * g + q]);
                bad |= !isfinite(to_f32(o[q]));
            }
            u32x2 st;
            st[0] = pack2(o[0], o[1]);
            st[1] = pack2(o[2], o[3]);
            *p = st;
        }
    };
    // one leaf, both row halves; its words are already issued into pre
    auto upd_pre = [&](int l, int b, int hf) {
        uint32_t uw[4][4];
        twait4<4>(pre, u_words(l, b, hf), wstr, a.tag0 + (uint32_t)l, uw, flags);
#pragma unroll
        for (int fn = 0; fn < 2; ++fn) {
            f32x16 acc = zero16();
            upd_product(acc, l, fn, uw);
            upd_store(acc, b, hf, fn);
        }
    };
    // leaves 0 .. l1 - 1, both row halves, the next leaf's words requested
    // before this leaf's products
    auto upd_run = [&](int l1, int b, int hf) {
        f32x16 acc[2] = {zero16(), zero16()};
        uint64_t vn[4][4];
        if (0 < l1) tissue4<4>(u_words(0, b, hf), wstr, vn);
        for (int l = 0; l < l1; ++l) {
            uint32_t uw[4][4];
            twait4<4>(vn, u_words(l, b, hf), wstr, a.tag0 + (uint32_t)l, uw, flags);
            if (l + 1 < l1) tissue4<4>(u_words(l + 1, b, hf), wstr, vn);
            upd_product(acc[0], l, 0, uw);
            upd_product(acc[1], l, 1, uw);
        }
        upd_store(acc[0], b, hf, 0);
        upd_store(acc[1], b, hf, 1);
    };
    // one leaf, one row half (the same sums in the same order), so that four
    // waves share a block
    auto upd_half = [&](int l, int b, int hf, int fn) {
        uint32_t uw[4][4];
        tfetch4<4>(u_words(l, b, hf), wstr, a.tag0 + (uint32_t)l, uw, flags);
        f32x16 acc = zero16();
        upd_product(acc, l, fn, uw);
        upd_store(acc, b, hf, fn);
    };
    // ---- the leaves above this tile: L tile, then the rank-64 update of the
    // blocks up to r + 1 only, block r + 1 one leaf behind (the last leaf,
    // r - 1, then updates the diagonal block beside leaf r - 2's update of
    // block r + 1).  Blocks further right take all their updates at once, with
    // one rounding, just before their U rows are formed.
    // A leaf forms its U rows in the order of the block columns, and this
    // workgroup has to be back for leaf r - 1 in time, so of leaf r - 2 it may
    // need the first two only.  Those must come soon: a run over all leaves
    // takes 1.4 us each (a memory round trip), so the sums of blocks r + 2 and
    // r + 3 are carried along in registers, a quarter block per wave and two
    // leaves behind, whose words are long there; the last leaves are added
    // after the hand-over.  Without these the chain waited on U rows from the
    // sixth leaf on, 20 us a leaf for 16.
    const int db = r + 2 + (w >> 2), dhf = (w >> 1) & 1, dfn = w & 1;
    const bool dac = db < nl;
    const int dl = std::max(r - 3, 0);  // leaves already in dacc after the loop
    f32x16 dacc = zero16();
    for (int l = 0; l < r; ++l) {
        const bool dstep = dac && l >= 2 && l - 2 < dl;
        const bool lstep = l == r - 1 && l > 0 && r + 1 < nl && w >= 4;
        if (dstep) tissue4<4>(u_words(l - 2, db, dhf), wstr, pre);
        if (lstep) tissue4<4>(u_words(l - 1, r + 1, dhf), wstr, pre);
        l21(l);
        // blocks l + 1 .. r by leaf l, then block r + 1 by leaf l - 1: four
        // units per block (column half, row half) where that leaves no wave
        // idle, else two, so that each word is fetched once
        const int nb = r - l, lag = l > 0 && r + 1 < nl ? 1 : 0;
        if (nb == 1) {
            if (w < 4) {
                upd_half(l, r, dhf, dfn);
            } else if (lstep) {
                uint32_t uw[4][4];
                twait4<4>(pre, u_words(l - 1, r + 1, dhf), wstr, a.tag0 + (uint32_t)(l - 1), uw, flags);
                f32x16 acc = zero16();
                upd_product(acc, l - 1, dfn, uw);
                upd_store(acc, r + 1, dhf, dfn);
            }
        } else if (nb == 2) {
            for (int u = w; u < 4 * (nb + lag); u += 8) {
                const bool late = u >= 4 * nb;
                upd_half(late ? l - 1 : l, late ? r + 1 : l + 1 + (u >> 2), (u >> 1) & 1, u & 1);
            }
        } else {
            for (int u = w; u < 2 * (nb + lag); u += 8) {
                const bool late = u >= 2 * nb;
                const int ll = late ? l - 1 : l, b = late ? r + 1 : l + 1 + (u >> 1), hf = u & 1;
                uint32_t uw[4][4];
                tfetch4<4>(u_words(ll, b, hf), wstr, a.tag0 + (uint32_t)ll, uw, flags);
#pragma unroll
                for (int fn = 0; fn < 2; ++fn) {
                    f32x16 acc = zero16();
                    upd_product(acc, ll, fn, uw);
                    upd_store(acc, b, hf, fn);
                }
            }
        }
        if (dstep) {
            uint32_t uw[4][4];
            twait4<4>(pre, u_words(l - 2, db, dhf), wstr, a.tag0 + (uint32_t)(l - 2), uw, flags);
            upd_product(dacc, l - 2, dfn, uw);
        }
        __syncthreads();
    }

    // the words of U(r - 1, r + 1), half w, that waves 0 and 1 apply to
    // block r + 1 right after the inversion (requested before the inversion)
    const bool have_pre = r > 0 && r + 1 < nl && w < 2;

    // ---- leaf r: factor the diagonal block (columns 64 r .. 64 r + 63) with
    // the partial-pivoting check.  Wave w keeps columns 8 w .. 8 w + 7 of all
    // 64 rows (lane = row); the owner of strip p factors it with readlane
    // broadcasts, and after one barrier every later wave applies it.
    {
        float x[8];
        {
            const u32x4 v = *(const u32x4 *)&tile[tix(lane, 64 * r + 8 * w, W)];
#pragma unroll
            for (int c = 0; c < 8; ++c) x[c] = to_f32(from_bits<T>(v[c >> 1] >> (16 * (c & 1))));
        }
        bool fail = false;
        // (unrolled: constant lanes in the broadcasts; 6.6 against 8.5 us)
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            if (w == p) {
#pragma unroll
                for (int kk = 0; kk < 8; ++kk) {
                    const int k = 8 * p + kk;
                    const float piv = lane_bcast(x[kk], k);
                    const float rp = rcp_nr(piv);
                    const bool below = lane > k;
                    fail |= !(fabsf(piv) > 0.0f) || (below && !(fabsf(x[kk]) <= margin * fabsf(piv)));
                    const float lx = x[kk] * rp;
                    const float lv = below ? lx : 0.0f;
                    x[kk] = below ? lx : x[kk];
                    // all broadcasts first, then the updates: independent
                    // readlanes issue back to back instead of alternating
                    // with the FMAs that consume them
                    float ub[8];
#pragma unroll
                    for (int c = kk + 1; c < 8; ++c) ub[c] = lane_bcast(x[c], k);
#pragma unroll
                    for (int c = kk + 1; c < 8; ++c) x[c] -= lv * ub[c];
                }
#pragma unroll
                for (int c = 0; c < 8; ++c) Dm[lane][8 * p + c] = x[c];
            }
            __syncthreads();
            if (w > p) {
                float lv[8];
#pragma unroll
                for (int kk = 0; kk < 8; ++kk) lv[kk] = lane > 8 * p + kk ? Dm[lane][8 * p + kk] : 0.0f;
#pragma unroll
                for (int kk = 0; kk < 8; ++kk) {
                    float ub[8];
#pragma unroll
                    for (int c = 0; c < 8; ++c) ub[c] = lane_bcast(x[c], 8 * p + kk);
#pragma unroll
                    for (int c = 0; c < 8; ++c) x[c] -= lv[kk] * ub[c];
                }
            }
        }
        if (fail) sfail = 1;
    }
    __syncthreads();
    if (t == 0 && sfail) set_flag(&flags[FLAG_FAIL], 1);
    // factored block into the tile (its final values)
    {
        const int i = t >> 3, cc = (t & 7) * 8;
        T o[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            o[q] = (T)Dm[i][cc + q];
            bad |= !isfinite(to_f32(o[q]));
        }
        u32x4 st;
#pragma unroll
        for (int p = 0; p < 4; ++p) st[p] = pack2(o[2 * p], o[2 * p + 1]);
        *(u32x4 *)&tile[tix(i, 64 * r + cc, W)] = st;
    }

    // U(r - 1, r + 1) requested now: leaf r - 1 forms it after handing over
    // U(r - 1, r), so a request before the diagonal factorisation could
    // still find the words unpublished and the wait after the inversion
    // would pay a whole round trip; requested here, the words are back with
    // the right tag by then and their latency is off the chain
    if (have_pre)
        tissue4<4>(a.pub + (size_t)(r - 1) * PUB_LEAF + PUB_U12 + (r + 1) * 2048 + op_word(w, 0, h, l32, 0),
                   op_word(0, 1, 0, 0, 0), pre);
    // the triangular inverses, and the scale exponents for their split into
    // halves from the largest entries (waves 0..3 U^{-1}, 4..7 L^{-1}, whose
    // unit diagonal is not stored)
    float mx = w < 4 ? 0.0f : 1.0f;
    mx = fmaxf(mx, inv_diag16(Dm, w, lane));
    __syncthreads();
    mx = fmaxf(mx, inv_double<16>(Dm, w, lane));
    __syncthreads();
    mx = wave_max(fmaxf(mx, inv_double<32>(Dm, w, lane)));
    if (lane == 0) red[w] = mx;
    __syncthreads();
    const int su = scale_exp(fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3])));
    const int sl = scale_exp(fmaxf(fmaxf(red[4], red[5]), fmaxf(red[6], red[7])));
    // ---- what leaf r passes on.  U(r, r + 1) first, since the next leaf's
    // workgroup waits for it: waves 0 and 1 form it with the scaled halves of
    // L^{-1} in registers, while waves 2..7 publish (U^{-1})^T (scaled
    // halves; row j of the operand is column j of U^{-1}) and write the same
    // words to the side buffer.  Then L^{-1} replaces Dm in LDS as the A
    // operand of the remaining U row blocks.
    T *iv = (T *)a.inv + (size_t)r * IH_LEAF;
    const float ful = ldexpf(1.0f, -sl);
    // U rows of leaf r in block columns b > r: U12 = L^{-1} T_b.  Unit
    // (b, fn): 32 columns of block b, both row halves.  A operand opa(fm, ks,
    // lo): the high (lo = 0) or low part of L^{-1} (rows 32 fm + l32) scaled
    // by 2^sl; B operand: 8 consecutive tile rows of one column.
    auto u12 = [&](int b, int fn, auto opa) {
        const uint32_t tag = a.tag0 + (uint32_t)r;
        uint64_t *pw = a.pub + (size_t)r * PUB_LEAF + PUB_U12 + b * 2048;
        const int c = 64 * b + 32 * fn + l32;
        vec tb[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            u32x4 v;
#pragma unroll
            for (int p = 0; p < 4; ++p)
                v[p] = pack2(tile[tix(16 * ks + 8 * h + 2 * p, c, W)], tile[tix(16 * ks + 8 * h + 2 * p + 1, c, W)]);
            tb[ks] = as_vec<T>(v);
        }
#pragma unroll
        for (int fm = 0; fm < 2; ++fm) {
            f32x16 acc = zero16();
#pragma unroll
            for (int ks = 0; ks < 2 + 2 * fm; ++ks) {  // L^{-1} is zero beyond
                acc = pmma<T>::op(opa(fm, ks, 0), tb[ks], acc);
                acc = pmma<T>::op(opa(fm, ks, 1), tb[ks], acc);
            }
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                T o[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    o[q] = (T)(acc[4 * g + q] * ful);
                    bad |= !isfinite(to_f32(o[q]));
                    tile[tix(32 * fm + 8 * g + 4 * h + q, c, W)] = o[q];
                }
                // rows k = 32 fm + 8 g + 4 h .. + 3 of operand row 32 fn + l32
                const int wd = op_word(fn, 2 * fm + (g >> 1), g & 1, l32, 2 * h);
                tstore(pw + wd, tag, pack2(o[0], o[1]));
                tstore(pw + wd + 1, tag, pack2(o[2], o[3]));
            }
        }
    };
    // the scaled L^{-1} operand piece (fm, ks) of this lane, from Dm
    auto linv8 = [&](int fm, int ks, vec &hi, vec &lo) {
        const float fl = ldexpf(1.0f, sl);
        const int m = 32 * fm + l32;
        float v[8];
        // every entry read (the address is always in the block), then the
        // triangle selected, so the reads are not masked one by one
#pragma unroll
        for (int p = 0; p < 8; ++p) v[p] = Dm[m][16 * ks + 8 * h + p];
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            const int k = 16 * ks + 8 * h + p;
            v[p] = (k < m ? v[p] : (k == m ? 1.0f : 0.0f)) * fl;
        }
        split8<T>(v, hi, lo);
    };
    if (w < 2) {
        if (r + 1 < nl) {
            vec lah[2][4], lal[2][4];
#pragma unroll
            for (int fm = 0; fm < 2; ++fm)
#pragma unroll
                for (int ks = 0; ks < 2 + 2 * fm; ++ks) linv8(fm, ks, lah[fm][ks], lal[fm][ks]);
            if (r > 0) upd_pre(r - 1, r + 1, w);
            u12(r + 1, w, [&](int fm, int ks, int lo) { return lo ? lal[fm][ks] : lah[fm][ks]; });
        }
    } else {
        const uint32_t tag = a.tag0 + (uint32_t)r;
        uint64_t *pr = a.pub + (size_t)r * PUB_LEAF;
        const float fu = ldexpf(1.0f, su);
        for (int x = t - 128; x < 1536; x += TOP_THREADS - 128) {  // the words that are not all zero
            const int e = x < 512 ? x : x + 512;                   // = op_word(fm, ks, h, l32, q)
            const int q = e & 3, l32e = (e >> 2) & 31, he = (e >> 7) & 1, kse = (e >> 8) & 3, fme = e >> 10;
            const int j = 32 * fme + l32e, k = 16 * kse + 8 * he + 2 * q;
            const float v0 = k <= j ? Dm[k][j] * fu : 0.0f;
            const float v1 = k + 1 <= j ? Dm[k + 1][j] * fu : 0.0f;
            const T h0 = (T)v0, h1 = (T)v1;
            const T q0 = (T)(v0 - to_f32(h0)), q1 = (T)(v1 - to_f32(h1));
            tstore(pr + PUB_UINV + e, tag, pack2(h0, h1));
            tstore(pr + PUB_UINV + 2048 + e, tag, pack2(q0, q1));
            *(uint32_t *)(iv + IH_UHI + 2 * e) = pack2(h0, h1);
            *(uint32_t *)(iv + IH_ULO + 2 * e) = pack2(q0, q1);
        }
        if (t - 128 < 4) tstore(pr + PUB_SCALE + (t - 128), tag, (uint32_t)su);
    }
    // L^{-1} to the side buffer and into LDS in place of Dm: wave w forms
    // step ks = w & 3 of row half fm = w >> 2
    u32x4 *lop = (u32x4 *)Dm;  // [hi / lo][fm][ks][lane]
    {
        vec hi, lo;
        linv8(w >> 2, w & 3, hi, lo);
        const u32x4 uhv = __builtin_bit_cast(u32x4, hi), ulv = __builtin_bit_cast(u32x4, lo);
        *(u32x4 *)(iv + IH_LHI + (w * 64 + lane) * 8) = uhv;
        *(u32x4 *)(iv + IH_LLO + (w * 64 + lane) * 8) = ulv;
        __syncthreads();  // every read of Dm done
        // the words of U^{-1} that are zero: for k_trsm only
        *(uint32_t *)(iv + IH_UHI + 2 * (512 + t)) = 0;
        *(uint32_t *)(iv + IH_ULO + 2 * (512 + t)) = 0;
        lop[w * 64 + lane] = uhv;
        lop[512 + w * 64 + lane] = ulv;
        if (t == 0) {
            int *ex = (int *)((T *)a.inv + IH_EXP);
            ex[2 * r] = su;
            ex[2 * r + 1] = sl;
        }
        __syncthreads();
    }
    // the carried blocks: their last leaves, then their U rows, block r + 2
    // first (after the barriers above, so that this does not slow the waves
    // that form U(r, r + 1): 3.4 against 2.7 us)
    auto opl = [&](int fm, int ks, int lo) { return as_vec<T>(lop[lo * 512 + (fm * 4 + ks) * 64 + lane]); };
    auto carried = [&]() {
        if (!dac || r == 0) return;
        for (int l = dl; l < r; ++l) {
            uint32_t uw[4][4];
            tfetch4<4>(u_words(l, db, dhf), wstr, a.tag0 + (uint32_t)l, uw, flags);
            upd_product(dacc, l, dfn, uw);
        }
        upd_store(dacc, db, dhf, dfn);
    };
    if (w < 4) carried();
    __syncthreads();
    if (w >= 4) carried();
    else if (w < 2 && r + 2 < nl) u12(r + 2, w, opl);
    __syncthreads();
    // the remaining U row blocks, 32 columns (unit j) per wave: block r + 3,
    // then block by block after their remaining updates (every leaf above at
    // once)
    for (int j = w; j < 2 * (nl - r - 3); j += 8) {
        const int b = r + 3 + (j >> 1), hf = j & 1;
        if (r > 0 && j >= 2) upd_run(r, b, hf);
        u12(b, hf, opl);
    }
    __syncthreads();

    // ---- copies of this row tile's off-diagonal blocks in operand order for
    // k_trsm: U(r, b)^T for b > r (element (m, k) = tile(k, 64 b + m)) and
    // L(r, i) for i < r (element (m, k) = tile(m, 64 i + k))
    {
        T *op = (T *)a.inv;
        for (int e = t; e < (nl - r - 1) * 512; e += TOP_THREADS) {
            const int b = r + 1 + e / 512, q = e % 512;
            const int ln = q & 63, fk = q >> 6;
            const int m = 32 * (fk >> 2) + (ln & 31), k = 16 * (fk & 3) + 8 * (ln >> 5);
            u32x4 v;
#pragma unroll
            for (int p = 0; p < 4; ++p)
                v[p] = pack2(tile[tix(k + 2 * p, 64 * b + m, W)], tile[tix(k + 2 * p + 1, 64 * b + m, W)]);
            *(u32x4 *)(op + OP_U + (size_t)(r * 16 + b) * 4096 + q * 8) = v;
        }
        for (int e = t; e < r * 512; e += TOP_THREADS) {
            const int i = e / 512, q = e % 512;
            const int ln = q & 63, fk = q >> 6;
            const int m = 32 * (fk >> 2) + (ln & 31), k = 16 * (fk & 3) + 8 * (ln >> 5);
            *(u32x4 *)(op + OP_L + (size_t)(r * 16 + i) * 4096 + q * 8) =
                *(const u32x4 *)&tile[tix(m, 64 * i + k, W)];
        }
    }
    // ---- the finished tile to A (column-major) and LT (row-major)
    for (int e = t; e < W * 8; e += TOP_THREADS) {
        const int c = e >> 3, rc = e & 7;
        u32x4 v;
#pragma unroll
        for (int p = 0; p < 4; ++p)
            v[p] = pack2(tile[tix(rc * 8 + 2 * p, c, W)], tile[tix(rc * 8 + 2 * p + 1, c, W)]);
        *(u32x4 *)(A + (row0 + rc * 8) + (k0 + c) * lda) = v;
    }
    {
        T *LT = (T *)a.LT;
        const int cpr = W / 8;
        for (int e = t; e < PT * cpr; e += TOP_THREADS) {
            const int i = e / cpr, cc = (e % cpr) * 8;
            *(u32x4 *)(LT + (row0 + i) * NB_OUT + cc) = *(const u32x4 *)&tile[tix(i, cc, W)];
        }
    }
    if (bad) set_flag(&flags[FLAG_NONFINITE], 1);
}

template <typename T>
__global__ __launch_bounds__(TOP_THREADS) void k_top(TopArgs a)
{
    __shared__ __attribute__((aligned(16))) char lds[TOP_LDS_BYTES];
    top_body<T>(a, blockIdx.x, lds);
}

// The next block's diagonal square and the rest of this block's trailing
// update in one launch: workgroups 0 .. ntop - 1 factor the square (they are
// dispatched first, on an idle device, so they are resident together), the
// others each take one 256x256 tile of C[M x N] -= At^T B (K = the block
// width).  The two touch disjoint data: the square's columns are left of
// the update's, and the square's L rows go to the other L buffer.
struct TopGemmArgs {
    TopArgs top;
    int ntop;
    int M, N, K;
    const void *At;
    int64_t ldat;
    const void *B;
    int64_t ldb;
    void *C;
    int64_t ldc;
    // a second region with the same K and leading dimensions (M2 = 0: none)
    int M2, N2;
    const void *At2;
    const void *B2;
    void *C2;
};

template <typename T>
__global__ __launch_bounds__(TOP_THREADS) void k_top_gemm(TopGemmArgs a)
{
    __shared__ __attribute__((aligned(16))) char lds[TOP_LDS_BYTES];
    static_assert(gemm16_lds_elems<256, 256, 32>() * 2 <= TOP_LDS_BYTES, "GEMM tile LDS");
    if ((int)blockIdx.x < a.ntop) {
        top_body<T>(a.top, blockIdx.x, lds);
        return;
    }
    if (block_flag(&a.top.flags[FLAG_FAIL])) return;
    const int ntm = a.M / 256, ntn = a.N / 256, n1 = ntm * ntn;
    const int ntm2 = a.M2 / 256, ntn2 = a.N2 / 256;
    int tile = xcd_tile((int)blockIdx.x - a.ntop, n1 + ntm2 * ntn2), tm, tn;
    if (tile < n1) {
        grouped_tile(tile, ntm, ntn, tm, tn);
        gemm16_tile<T, 256, 256, 2, 4, 32>(tm * 256, tn * 256, a.K, (const T *)a.At, a.ldat,
                                           (const T *)a.B, a.ldb, (T *)a.C, a.ldc, a.top.flags, (T *)lds);
    } else {
        grouped_tile(tile - n1, ntm2, ntn2, tm, tn);
        gemm16_tile<T, 256, 256, 2, 4, 32>(tm * 256, tn * 256, a.K, (const T *)a.At2, a.ldat,
                                           (const T *)a.B2, a.ldb, (T *)a.C2, a.ldc, a.top.flags, (T *)lds);
    }
}

// ====================================================================== k_trsm
struct TrsmArgs {
    int64_t k0;
    int W;
    int nrt;          // 64-row tiles below the square (= 64-column slabs right of it)
    void *A;
    int64_t lda;
    void *LT;
    const void *inv;  // the inverses' side buffer written by k_top
    int *flags;
};

// Element (k, c) of a slab of 64 columns with columns of R values held
// column-major in LDS; chunks of 8 rows permuted by XOR with c & 7.
__device__ __forceinline__ int six(int k, int c, int R)
{
    return c * R + ((((k >> 3) ^ (c & 7)) << 3) | (k & 7));
}

// Per-workgroup state of k_trsm.  Eight wavefronts; wave w takes the 32x32
// fragment f = w & 3 ((fm, fn) = (f & 1, f >> 1)) of each 64x64 block and
// one half kh = w >> 2 of the K range of its sum.  Left-looking: block I's
// sum over the finished blocks i < I (U(i,I)^T L(:,i)^T for the rows below,
// L(I,i) U(i) for the columns right) is formed in FP32 at step I, so every
// entry is rounded to the storage type once.  The global operands of step
// I + 1's sum are requested as soon as step I's sum has consumed its
// registers, so their latency overlaps step I's diagonal-block work; waves
// 0..3 then solve the block (one fragment each).
// A block is a chain of four barriers (halves joined, largest entry, staged
// operands, block stored); with the inverse's operands requested by all eight
// waves at the head of the block, and six barriers, 256 workgroups took 74 us
// instead of 70 (4.4 us a block) and 480 (two rounds) 159 instead of 150.
constexpr int TRSM_PF = 2 * (NB_OUT / PT - 1);  // 16-deep K steps of the longest half sum

template <typename T> struct TrsmCtx {
    int64_t k0, lda, base;   // base: first row (role L) or column (role U) of the 64
    int W, nl, w, kh, h, l32, fm, fn;
    T *A;
    const T *LT, *inv;
    int ex[32];              // the leaves' exponents (s of U^{-1}, s of L^{-1})
    T *buf, *sth, *stl;      // the tile; the staged high and low parts of one block
    float *pbuf;             // the K halves' hand-over, 16 x 64 values per fragment
    bool bad, fail;
};

// the scaled high/low split of the FP32 values y (this lane's 16 fragment
// entries, waves 0..3) staged for use as a matrix-core operand; returns the
// exponent
template <typename T>
__device__ __forceinline__ int stage_split(TrsmCtx<T> &c, const float (&y)[16], bool rowmajor)
{
    float mx = 0.0f;
#pragma unroll
    for (int q = 0; q < 16; ++q) mx = fmaxf(mx, fabsf(y[q]));
    // the four maxima cross through the head of each wavefront's own part of
    // pbuf, which it has read (join_halves); they are read before the barrier
    // that follows this function, and waves 4..7 write pbuf again in the next
    // block's join_halves, which they enter after this block's last barrier
    mx = wave_max(mx);
    if (c.w < 4 && (threadIdx.x & 63) == 0) c.pbuf[c.w * 1024] = mx;
    __syncthreads();
    if (c.w >= 4) return 0;
    const int sy = scale_exp(fmaxf(fmaxf(c.pbuf[0], c.pbuf[1024]), fmaxf(c.pbuf[2048], c.pbuf[3072])));
    const float fy = ldexpf(1.0f, sy);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        T hi[4], lo[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float v = y[4 * g + q] * fy;
            hi[q] = (T)v;
            lo[q] = (T)(v - to_f32(hi[q]));
        }
        u32x2 sh, sl;
        sh[0] = pack2(hi[0], hi[1]);
        sh[1] = pack2(hi[2], hi[3]);
        sl[0] = pack2(lo[0], lo[1]);
        sl[1] = pack2(lo[2], lo[3]);
        const int k = 32 * c.fm + 8 * g + 4 * c.h;  // fragment row (block-local)
        if (rowmajor) {  // role L: entry (tile row i, leaf column k)
            const int i = 32 * c.fn + c.l32;
            *(u32x2 *)&c.sth[tix(i, k, PT)] = sh;
            *(u32x2 *)&c.stl[tix(i, k, PT)] = sl;
        } else {         // role U: entry (block row k, slab column cc)
            const int cc = 32 * c.fn + c.l32;
            *(u32x2 *)&c.sth[six(k, cc, PT)] = sh;
            *(u32x2 *)&c.stl[six(k, cc, PT)] = sl;
        }
    }
    return sy;
}

// the two K halves of a fragment's sum: waves 4..7 hand theirs to waves 0..3
template <typename T>
__device__ __forceinline__ void join_halves(TrsmCtx<T> &c, f32x16 &p)
{
    const int lane = 32 * c.h + c.l32, f = c.w & 3;
    if (c.kh == 1) {
#pragma unroll
        for (int j = 0; j < 16; ++j) c.pbuf[(f * 16 + j) * 64 + lane] = p[j];
    }
    __syncthreads();
    if (c.kh == 0) {
#pragma unroll
        for (int j = 0; j < 16; ++j) p[j] += c.pbuf[(f * 16 + j) * 64 + lane];
    }
}

// ---- role L, block I: L(:, I) = (X_I - sum_{i<I} L(:, i) U(i, I)) U_II^{-1}.
// pf: this wave's A operands of block I's half sum (requested at step I - 1).
template <typename T, int I> struct StepL {
    typedef typename pmma<T>::vec vec;
    static __device__ __forceinline__ void prefetch(const TrsmCtx<T> &c, u32x4 (&pf)[TRSM_PF])
    {
        if constexpr (I >= 1 && I < 16) {
            if (I < c.nl) {
                const T *op = c.inv + OP_U + I * 4096 + (c.fm * 4 * 64 + 32 * c.h + c.l32) * 8;
#pragma unroll
                for (int s = 0; s < 2 * I; ++s) {
                    const int K = c.kh * 32 * I + 16 * s;  // block K >> 6, step (K >> 4) & 3
                    pf[s] = *(const u32x4 *)(op + (K >> 6) * 16 * 4096 + ((K >> 4) & 3) * 64 * 8);
                }
            }
        }
    }
    static __device__ __forceinline__ void run(TrsmCtx<T> &c, u32x4 (&pf)[TRSM_PF])
    {
        if (I >= c.nl) return;
        const int W = c.W, h = c.h, l32 = c.l32, fm = c.fm, fn = c.fn;
        const int i = 32 * fn + l32;
        // this wave's half of P^T = U(<I, I)^T L(:, <I)^T
        f32x16 p = zero16();
#pragma unroll
        for (int s = 0; s < 2 * I; ++s) {
            const vec bv = as_vec<T>(*(const u32x4 *)&c.buf[tix(i, c.kh * 32 * I + 16 * s + 8 * h, W)]);
            p = pmma<T>::op(as_vec<T>(pf[s]), bv, p);
        }
        // the inverse's operands (waves 0..3), then the next block's: in this
        // order, so that the wait for these does not wait for those
        u32x4 uh[4], ul[4];
        if (c.w < 4) {
            const T *iv = c.inv + (size_t)I * IH_LEAF + (fm * 4 * 64 + 32 * h + l32) * 8;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                uh[ks] = *(const u32x4 *)(iv + IH_UHI + ks * 64 * 8);
                ul[ks] = *(const u32x4 *)(iv + IH_ULO + ks * 64 * 8);
            }
        }
        StepL<T, I + 1>::prefetch(c, pf);
        join_halves(c, p);
        // Y^T fragment: rows = leaf columns 32 fm + 8 g + 4 h + q of block I, column = tile row i
        float y[16];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const u32x2 xv = *(const u32x2 *)&c.buf[tix(i, 64 * I + 32 * fm + 8 * g + 4 * h, W)];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                y[4 * g + q] = to_f32(from_bits<T>(xv[q >> 1] >> (16 * (q & 1)))) - p[4 * g + q];
        }
        const int sy = stage_split<T>(c, y, true);
        __syncthreads();
        f32x16 r = zero16();
        if (c.w < 4) {
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const vec yh = as_vec<T>(*(const u32x4 *)&c.sth[tix(i, 16 * ks + 8 * h, PT)]);
                const vec yl = as_vec<T>(*(const u32x4 *)&c.stl[tix(i, 16 * ks + 8 * h, PT)]);
                r = pmma<T>::op(as_vec<T>(uh[ks]), yh, r);
                r = pmma<T>::op(as_vec<T>(ul[ks]), yh, r);
                r = pmma<T>::op(as_vec<T>(uh[ks]), yl, r);
            }
        }
        if (c.w < 4) {
            const float back = ldexpf(1.0f, -(c.ex[2 * I] + sy));
            const float margin = 1.0f - 1.0f / 256.0f;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                T o[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float v = r[4 * g + q] * back;
                    c.fail |= !(fabsf(v) <= margin);
                    o[q] = (T)v;
                }
                u32x2 st;
                st[0] = pack2(o[0], o[1]);
                st[1] = pack2(o[2], o[3]);
                *(u32x2 *)&c.buf[tix(i, 64 * I + 32 * fm + 8 * g + 4 * h, W)] = st;
            }
        }
        __syncthreads();
        StepL<T, I + 1>::run(c, pf);
    }
};
template <typename T> struct StepL<T, 16> {
    static __device__ __forceinline__ void prefetch(const TrsmCtx<T> &, u32x4 (&)[TRSM_PF]) {}
    static __device__ __forceinline__ void run(TrsmCtx<T> &, u32x4 (&)[TRSM_PF]) {}
};

// ---- role U, block row I: U_I = L_II^{-1} (A_I - sum_{m<I} L(I, m) U_m).
template <typename T, int I> struct StepU {
    typedef typename pmma<T>::vec vec;
    static __device__ __forceinline__ void prefetch(const TrsmCtx<T> &c, u32x4 (&pf)[TRSM_PF])
    {
        if constexpr (I >= 1 && I < 16) {
            if (I < c.nl) {
                const T *op = c.inv + OP_L + I * 16 * 4096 + (c.fm * 4 * 64 + 32 * c.h + c.l32) * 8;
#pragma unroll
                for (int s = 0; s < 2 * I; ++s) {
                    const int K = c.kh * 32 * I + 16 * s;  // block K >> 6, step (K >> 4) & 3
                    pf[s] = *(const u32x4 *)(op + (K >> 6) * 4096 + ((K >> 4) & 3) * 64 * 8);
                }
            }
        }
    }
    static __device__ __forceinline__ void run(TrsmCtx<T> &c, u32x4 (&pf)[TRSM_PF])
    {
        if (I >= c.nl) return;
        const int W = c.W, h = c.h, l32 = c.l32, fm = c.fm, fn = c.fn;
        const int cc = 32 * fn + l32;  // slab column of this lane
        T *acol = c.A + (c.k0 + 64 * I + 32 * fm) + (c.base + cc) * c.lda;
        u32x2 xa[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) xa[g] = *(const u32x2 *)(acol + 8 * g + 4 * h);
        // this wave's half of P = L(I, <I) U(<I)
        f32x16 p = zero16();
#pragma unroll
        for (int s = 0; s < 2 * I; ++s) {
            const vec bv = as_vec<T>(*(const u32x4 *)&c.buf[six(c.kh * 32 * I + 16 * s + 8 * h, cc, W)]);
            p = pmma<T>::op(as_vec<T>(pf[s]), bv, p);
        }
        // the inverse's operands (waves 0..3), then the next block's: in this
        // order, so that the wait for these does not wait for those
        u32x4 lh[4], ll[4];
        if (c.w < 4) {
            const T *iv = c.inv + (size_t)I * IH_LEAF + (fm * 4 * 64 + 32 * h + l32) * 8;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                lh[ks] = *(const u32x4 *)(iv + IH_LHI + ks * 64 * 8);
                ll[ks] = *(const u32x4 *)(iv + IH_LLO + ks * 64 * 8);
            }
        }
        StepU<T, I + 1>::prefetch(c, pf);
        join_halves(c, p);
        // Z fragment: rows 32 fm + 8 g + 4 h + q of block row I, column cc
        float z[16];
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                z[4 * g + q] = to_f32(from_bits<T>(xa[g][q >> 1] >> (16 * (q & 1)))) - p[4 * g + q];
        const int sz = stage_split<T>(c, z, false);
        __syncthreads();
        f32x16 r = zero16();
        if (c.w < 4) {
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const vec zh = as_vec<T>(*(const u32x4 *)&c.sth[six(16 * ks + 8 * h, cc, PT)]);
                const vec zl = as_vec<T>(*(const u32x4 *)&c.stl[six(16 * ks + 8 * h, cc, PT)]);
                r = pmma<T>::op(as_vec<T>(lh[ks]), zh, r);
                r = pmma<T>::op(as_vec<T>(ll[ks]), zh, r);
                r = pmma<T>::op(as_vec<T>(lh[ks]), zl, r);
            }
        }
        if (c.w < 4) {
            const float back = ldexpf(1.0f, -(c.ex[2 * I + 1] + sz));
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                T o[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    o[q] = (T)(r[4 * g + q] * back);
                    c.bad |= !isfinite(to_f32(o[q]));
                }
                u32x2 st;
                st[0] = pack2(o[0], o[1]);
                st[1] = pack2(o[2], o[3]);
                *(u32x2 *)&c.buf[six(64 * I + 32 * fm + 8 * g + 4 * h, cc, W)] = st;
                *(u32x2 *)(acol + 8 * g + 4 * h) = st;
            }
        }
        __syncthreads();
        StepU<T, I + 1>::run(c, pf);
    }
};
template <typename T> struct StepU<T, 16> {
    static __device__ __forceinline__ void prefetch(const TrsmCtx<T> &, u32x4 (&)[TRSM_PF]) {}
    static __device__ __forceinline__ void run(TrsmCtx<T> &, u32x4 (&)[TRSM_PF]) {}
};

template <typename T>
__global__ __launch_bounds__(TRSM_THREADS) void k_trsm(TrsmArgs a)
{
    __shared__ __attribute__((aligned(16))) T buf[PT * NB_OUT];
    __shared__ __attribute__((aligned(16))) T sth[PT * PT], stl[PT * PT];
    __shared__ float pbuf[4 * 16 * 64];  // with the above all of the 160 KB
    if (threadIdx.x == 0) pbuf[0] = __int_as_float(ld_flag(&a.flags[FLAG_FAIL]));
    __syncthreads();
    if (__float_as_int(pbuf[0])) return;  // block-uniform
    __syncthreads();
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int W = a.W;
    const int64_t k0 = a.k0, kend = k0 + W, lda = a.lda;
    T *A = (T *)a.A;
    TrsmCtx<T> c;
    c.k0 = k0;
    c.lda = lda;
    c.W = W;
    c.nl = W / PT;
    c.w = w;
    c.kh = w >> 2;
    c.fm = w & 1;
    c.fn = (w >> 1) & 1;
    c.h = lane >> 5;
    c.l32 = lane & 31;
    c.A = A;
    c.LT = (const T *)a.LT;
    c.inv = (const T *)a.inv;
    c.buf = buf;
    c.sth = sth;
    c.stl = stl;
    c.pbuf = pbuf;
    c.bad = false;
    c.fail = false;
    {
        const int *ex = (const int *)((const T *)a.inv + IH_EXP);
#pragma unroll
        for (int k = 0; k < 32; ++k) c.ex[k] = ex[k];
    }
    u32x4 pf[TRSM_PF];
    if ((int)blockIdx.x < a.nrt) {
        // ---- L rows of the tile [row0, row0 + 64)
        const int64_t row0 = kend + (int64_t)blockIdx.x * PT;
        c.base = row0;
        for (int e = t; e < W * 8; e += TRSM_THREADS) {
            const int col = e >> 3, rc = e & 7;
            const u32x4 v = *(const u32x4 *)(A + (row0 + rc * 8) + (k0 + col) * lda);
#pragma unroll
            for (int q = 0; q < 8; ++q) buf[tix(rc * 8 + q, col, W)] = from_bits<T>(v[q >> 1] >> (16 * (q & 1)));
        }
        __syncthreads();
        StepL<T, 0>::run(c, pf);
        for (int e = t; e < W * 8; e += TRSM_THREADS) {
            const int col = e >> 3, rc = e & 7;
            u32x4 v;
#pragma unroll
            for (int p = 0; p < 4; ++p)
                v[p] = pack2(buf[tix(rc * 8 + 2 * p, col, W)], buf[tix(rc * 8 + 2 * p + 1, col, W)]);
            *(u32x4 *)(A + (row0 + rc * 8) + (k0 + col) * lda) = v;
        }
        T *LT = (T *)a.LT;
        const int cpr = W / 8;
        for (int e = t; e < PT * cpr; e += TRSM_THREADS) {
            const int ii = e / cpr, cc = (e % cpr) * 8;
            *(u32x4 *)(LT + (row0 + ii) * NB_OUT + cc) = *(const u32x4 *)&buf[tix(ii, cc, W)];
        }
    } else {
        // ---- U rows of the slab [col0, col0 + 64); buf holds the slab's
        // finished U rows (column-major, W rows)
        c.base = kend + (int64_t)(blockIdx.x - a.nrt) * PT;
        StepU<T, 0>::run(c, pf);
    }
    if (c.fail) set_flag(&a.flags[FLAG_FAIL], 1);
    if (c.bad) set_flag(&a.flags[FLAG_NONFINITE], 1);
}

template <typename T>
hipError_t top_t(int64_t k0, int W, void *A, int64_t lda, void *LT, uint64_t *pub, float *inv,
                 int *flags, uint32_t tag0, hipStream_t s)
{
    TopArgs a{k0, W, A, lda, LT, pub, inv, flags, tag0};
    hipLaunchKernelGGL(k_top<T>, dim3((unsigned)(W / PT)), dim3(TOP_THREADS), 0, s, a);
    return hipGetLastError();
}

template <typename T>
hipError_t top_gemm_t(TopGemmArgs a, hipStream_t s)
{
    const unsigned grid = (unsigned)(a.ntop + (a.M / 256) * (a.N / 256) + (a.M2 / 256) * (a.N2 / 256));
    hipLaunchKernelGGL(k_top_gemm<T>, dim3(grid), dim3(TOP_THREADS), 0, s, a);
    return hipGetLastError();
}

template <typename T>
hipError_t trsm_t(int64_t k0, int W, int nrt, void *A, int64_t lda, void *LT, const float *inv,
                  int *flags, hipStream_t s)
{
    TrsmArgs a{k0, W, nrt, A, lda, LT, inv, flags};
    hipLaunchKernelGGL(k_trsm<T>, dim3((unsigned)(2 * nrt)), dim3(TRSM_THREADS), 0, s, a);
    return hipGetLastError();
}

}  // namespace

size_t top_pub_words() { return (size_t)PUB_LEAF * (NB_OUT / PT); }
size_t top_inv_floats() { return (size_t)IH_TOTAL * 2 / 4; }

hipError_t launch_top(int prec, int64_t k0, int W, void *A, int64_t lda, void *LT, uint64_t *pub,
                      float *inv, int *flags, uint32_t tag0, hipStream_t s)
{
    if (W < PT || W > NB_OUT || W % PT || lda % 8 || k0 % PT) return hipErrorInvalidValue;
    switch (prec) {
    case N3P_FP16: return top_t<f16>(k0, W, A, lda, LT, pub, inv, flags, tag0, s);
    case N3P_BF16: return top_t<bf16>(k0, W, A, lda, LT, pub, inv, flags, tag0, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_top_gemm(int prec, int64_t k0, int W, void *A, int64_t lda, void *LT,
                           uint64_t *pub, float *inv, int *flags, uint32_t tag0, int64_t M,
                           int64_t N, int64_t K, const void *At, int64_t ldat, const void *B,
                           int64_t ldb, void *C, int64_t ldc, int64_t M2, int64_t N2,
                           const void *At2, const void *B2, void *C2, hipStream_t s)
{
    if (W < PT || W > NB_OUT || W % PT || lda % 8 || k0 % PT) return hipErrorInvalidValue;
    if (M <= 0 || N <= 0 || M % 256 || N % 256 || K % 64 || K <= 0) return hipErrorInvalidValue;
    if (M2 < 0 || N2 < 0 || M2 % 256 || N2 % 256) return hipErrorInvalidValue;
    if (M2 == 0 || N2 == 0) M2 = N2 = 0;
    TopGemmArgs g{TopArgs{k0, W, A, lda, LT, pub, inv, flags, tag0}, W / PT, (int)M, (int)N, (int)K,
                  At, ldat, B, ldb, C, ldc, (int)M2, (int)N2, At2, B2, C2};
    switch (prec) {
    case N3P_FP16: return top_gemm_t<f16>(g, s);
    case N3P_BF16: return top_gemm_t<bf16>(g, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_trsm(int prec, int64_t Np, int64_t k0, int W, void *A, int64_t lda, void *LT,
                       const float *inv, int *flags, hipStream_t s)
{
    const int64_t rest = Np - k0 - W;
    if (rest <= 0) return hipSuccess;
    if (W < PT || W > NB_OUT || W % PT || rest % PT || lda % 8) return hipErrorInvalidValue;
    const int nrt = (int)(rest / PT);
    switch (prec) {
    case N3P_FP16: return trsm_t<f16>(k0, W, nrt, A, lda, LT, inv, flags, s);
    case N3P_BF16: return trsm_t<bf16>(k0, W, nrt, A, lda, LT, inv, flags, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace n3p
