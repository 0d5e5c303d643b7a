// k_getrf.hip -- blocked right-looking LU with partial pivoting for gfx950.
//
// The factorisation (Gaussian elimination, Section 1.3; the half-precision
// factorisation J_h = L U of Section 2) runs on the padded Np x Np copy:
//
//   for each outer block of NB_OUT columns (1024; sizes padded to 512):
//     for each leaf of NB_LEAF columns inside it:
//       leaf kernel   -- factor the leaf, form L21 and the U row block
//       inner GEMMs   -- update the rest of the outer block (K = NB_LEAF)
//     outer GEMM      -- Schur complement of the trailing matrix (K = NB_OUT)
//
// Pivoting: the leaf kernel first tries the diagonal as pivot and verifies,
// column by column, that every candidate below it is smaller in magnitude by
// a margin (|a_ij| <= (1 - 2^-8) |a_jj|).  When that holds for every column,
// partial pivoting (largest magnitude, ties to the lowest row) selects the
// diagonal at every step, so the no-interchange factorisation IS the
// partial-pivoting one.  If any column fails the test, a flag aborts the
// remaining kernels and the host re-runs the factorisation with explicit
// pivot searches and row interchanges (k_pivot.hip).  Near-ties
// always take the explicit path, so rounding differences cannot change a
// pivot decision.
//
// The Schur-complement GEMMs use the matrix cores: FP16/BF16 inputs with FP32
// accumulation (v_mfma_f32_32x32x16_{f16,bf16}), rounded to the storage type
// once per GEMM; FP32 and FP64 use v_mfma_{f32,f64}_16x16x4.
#include <algorithm>

#include "n3p_gemm.hpp"

namespace n3p {

// recip: 1/v.  FP32: hardware reciprocal estimate refined by one Newton-Raphson
// step (r + r(1 - v r)), within an ulp of the rounded quotient; FP64: division.
__device__ __forceinline__ float recip(float v)
{
    const float r = __builtin_amdgcn_rcpf(v);
    return fmaf(fmaf(-v, r, 1.0f), r, r);
}
__device__ __forceinline__ double recip(double v) { return 1.0 / v; }

// =========================================================== leaf (no-swap)
// Tile b < nrt: 64 rows of L21 below the leaf; nrt <= b < nrt + nct: 64
// columns of the U row block to the right of the leaf (when the leaf is the
// last one, a single tile only stores the diagonal block).  Every workgroup
// factors the 64x64 diagonal block itself (identical arithmetic in every
// workgroup), so none waits for another.  The factored diagonal block goes to
// DG (a side buffer): workgroups still reading the unfactored block from A
// must not see it change; with DG null (allowed only when the leaf has no
// tiles) it goes straight to A.  DGprev (if non-null) is the previous leaf's
// diagonal block, copied into A by tile 0 (nothing else touches that region
// now).  L21 is also written transposed to LT (row i at LT + i * ldlt + ltcol,
// K contiguous) for the Schur update.
//
// The chain of 64 column steps bounds the leaf, so the tile rides along it: a
// wavefront holds 8 columns of the diagonal block and of the L21 rows (or 8
// rows of the block and of the U12 columns), one row (column) per lane, and
// the broadcasts that eliminate the block serve the tile as well.  Panels of 8
// steps pass from wavefront to wavefront through LDS, one barrier each.  A
// solve of the tile after the block's factorisation cost another 10 us (its
// coefficients, 64 per lane and group of 8 steps, kept the LDS busy).  The
// panel loop is unrolled for constant lanes in the broadcasts (FP64: 20 -> 17
// us).  Measured: k_leaf_spec<double> 29.2 -> 17.1 us (2 and 92 tiles alike);
// the batched FP16 leaf 25.2 -> 18.4 us, 35 -> 32 us with four tiles a CU.
constexpr int LEAF_THREADS = 512;

// eight consecutive elements (16-byte aligned) to and from the compute type
template <typename T, typename CT> __device__ __forceinline__ void load8(const T *src, CT (&v)[8])
{
    typedef T vec __attribute__((ext_vector_type(16 / sizeof(T))));
    constexpr int CH = 16 / (int)sizeof(T);
#pragma unroll
    for (int q = 0; q < 8 / CH; ++q) {
        const vec e = *(const vec *)(src + q * CH);
#pragma unroll
        for (int u = 0; u < CH; ++u) v[q * CH + u] = (CT)to_f32((T)e[u]);
    }
}
template <typename T, typename CT> __device__ __forceinline__ void store8(T *dst, const CT (&v)[8])
{
    typedef T vec __attribute__((ext_vector_type(16 / sizeof(T))));
    constexpr int CH = 16 / (int)sizeof(T);
#pragma unroll
    for (int q = 0; q < 8 / CH; ++q) {
        vec e;
#pragma unroll
        for (int u = 0; u < CH; ++u) e[u] = to_store_d<T>((double)v[q * CH + u]);
        *(vec *)(dst + q * CH) = e;
    }
}

template <typename T>
__device__ __forceinline__ void leaf_body(int bid, int64_t Np, int64_t c0, T *__restrict__ A,
                                          int64_t lda, T *__restrict__ LT, int64_t ldlt,
                                          int64_t ltcol, int nrt, int nct, T *__restrict__ DG,
                                          const T *__restrict__ DGprev, int64_t cprev,
                                          int *__restrict__ flags)
{
    typedef typename compute_of<T>::type CT;
    constexpr int L = NB_LEAF, NT = LEAF_THREADS;
    // step k: the block's multipliers by row (its U row by column), and the
    // tile's L21 column (its U12 row)
    __shared__ CT Pm[L][L];
    __shared__ CT Zm[L][L];
    __shared__ CT rs[L];
    __shared__ int sfail, s_flag;
    const int t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    int fl = 0;
    if (t == 0) fl = ld_flag(&flags[FLAG_FAIL]);
    const CT margin = (CT)(1.0 - 1.0 / 256.0);
    bool bad = false;
    CT x[8], z[8];
    if (bid < nrt || nrt == 0) {
        // ---- 64 rows [R0, R0+64) of L21, lane = row.  Wave w keeps columns
        // 8w .. 8w+7 of the block (x) and of the tile (z); the pivot row's
        // entries come by readlane.  An entry of the tile is checked against
        // the pivot when its column is eliminated: the Schur complement entry
        // that partial pivoting would compare.
        const int64_t R0 = c0 + L + (int64_t)bid * L;
        const bool tile = bid < nrt;
        T dp[L * L / NT];
        if (bid == 0 && DGprev) {
#pragma unroll
            for (int q = 0; q < L * L / NT; ++q) dp[q] = DGprev[t + q * NT];
        }
        T *Dc = A + (c0 + lane) + (c0 + 8 * w) * lda, *Zc = A + (R0 + lane) + (c0 + 8 * w) * lda;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            x[c] = (CT)to_f32(Dc[c * lda]);
            z[c] = tile ? (CT)to_f32(Zc[c * lda]) : (CT)0;
        }
        if (t == 0) {
            s_flag = fl;
            sfail = 0;
        }
        bool fail = false, zfail = false;
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            if (w == p) {
#pragma unroll
                for (int kk = 0; kk < 8; ++kk) {
                    const int k = 8 * p + kk;
                    // branch-free (selects, no exec-mask branches), and every
                    // broadcast before the updates: this is the leaf's serial chain
                    const CT piv = lane_bcast(x[kk], k);
                    const CT rp = recip(piv);
                    const bool below = lane > k;
                    const CT lim = margin * fabs(piv);
                    fail |= !(fabs(piv) > (CT)0) || (below && !(fabs(x[kk]) <= lim));
                    zfail |= !(fabs(z[kk]) <= lim);
                    const CT lx = x[kk] * rp;
                    const CT l = below ? lx : (CT)0;
                    x[kk] = below ? lx : x[kk];
                    z[kk] *= (CT)1 / piv;
                    Pm[k][lane] = l;
                    Zm[k][lane] = z[kk];
                    CT ub[8];
#pragma unroll
                    for (int c = kk + 1; c < 8; ++c) ub[c] = lane_bcast(x[c], k);
#pragma unroll
                    for (int c = kk + 1; c < 8; ++c) {
                        x[c] -= l * ub[c];
                        z[c] -= z[kk] * ub[c];
                    }
                }
            }
            __syncthreads();
            if (p == 0 && s_flag) return;  // block-uniform
            if (w > p) {
                CT l[8], zl[8];
#pragma unroll
                for (int kk = 0; kk < 8; ++kk) {
                    l[kk] = Pm[8 * p + kk][lane];
                    zl[kk] = Zm[8 * p + kk][lane];
                }
#pragma unroll
                for (int kk = 0; kk < 8; ++kk) {
                    CT ub[8];
#pragma unroll
                    for (int c = 0; c < 8; ++c) ub[c] = lane_bcast(x[c], 8 * p + kk);
#pragma unroll
                    for (int c = 0; c < 8; ++c) {
                        x[c] -= l[kk] * ub[c];
                        z[c] -= zl[kk] * ub[c];
                    }
                }
            }
        }
        if (fail) sfail = 1;
        __syncthreads();
        if (sfail) {  // block-uniform: settled before the barrier
            if (t == 0) set_flag(&flags[FLAG_FAIL], 1);
            return;
        }
        if (bid == 0) {
            if (DGprev) {
#pragma unroll
                for (int q = 0; q < L * L / NT; ++q) {
                    const int e = t + q * NT;
                    A[(cprev + e % L) + (cprev + e / L) * lda] = dp[q];
                }
            }
            T *out = DG ? DG + lane + 8 * w * L : Dc;
            const int64_t ldo = DG ? L : lda;
#pragma unroll
            for (int c = 0; c < 8; ++c) out[c * ldo] = to_store_d<T>((double)x[c]);
        }
        if (!tile) return;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const T v = to_store_d<T>((double)z[c]);
            bad |= !isfinite(to_f32(v));  // the stored value
            Zc[c * lda] = v;
        }
        store8(LT + (R0 + lane) * ldlt + ltcol + 8 * w, z);
        if (zfail) set_flag(&flags[FLAG_FAIL], 1);
    } else {
        // ---- 64 columns [C0, C0+64) of U12, lane = column.  Wave w keeps
        // rows 8w .. 8w+7 of the block (x) and of the tile (z); the multiplier
        // of row i at step k is lane k's entry of that row over the pivot, the
        // same product as above.  The block is checked by the L21 tiles.
        const int64_t C0 = c0 + L + (int64_t)(bid - nrt) * L;
        load8(A + c0 + 8 * w + (c0 + lane) * lda, x);
        load8(A + c0 + 8 * w + (C0 + lane) * lda, z);
        if (t == 0) s_flag = fl;
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            if (w == p) {
#pragma unroll
                for (int kk = 0; kk < 8; ++kk) {
                    const int k = 8 * p + kk;
                    const CT rp = recip(lane_bcast(x[kk], k));
                    const CT u = lane > k ? x[kk] : (CT)0;
                    Pm[k][lane] = u;
                    Zm[k][lane] = z[kk];
                    if (lane == 0) rs[k] = rp;
                    CT l[8];
#pragma unroll
                    for (int c = kk + 1; c < 8; ++c) l[c] = lane_bcast(x[c], k) * rp;
#pragma unroll
                    for (int c = kk + 1; c < 8; ++c) {
                        x[c] -= l[c] * u;
                        z[c] -= l[c] * z[kk];
                    }
                }
            }
            __syncthreads();
            if (p == 0 && s_flag) return;  // block-uniform
            if (w > p) {
                CT u[8], zu[8], rk[8];
#pragma unroll
                for (int kk = 0; kk < 8; ++kk) {
                    u[kk] = Pm[8 * p + kk][lane];
                    zu[kk] = Zm[8 * p + kk][lane];
                    rk[kk] = rs[8 * p + kk];
                }
#pragma unroll
                for (int kk = 0; kk < 8; ++kk) {
                    CT l[8];
#pragma unroll
                    for (int c = 0; c < 8; ++c) l[c] = lane_bcast(x[c], 8 * p + kk) * rk[kk];
#pragma unroll
                    for (int c = 0; c < 8; ++c) {
                        x[c] -= l[c] * u[kk];
                        z[c] -= l[c] * zu[kk];
                    }
                }
            }
        }
        store8(A + c0 + 8 * w + (C0 + lane) * lda, z);
#pragma unroll
        for (int c = 0; c < 8; ++c) bad |= !isfinite(to_f32(to_store_d<T>((double)z[c])));
    }
    if (bad) set_flag(&flags[FLAG_NONFINITE], 1);
}

template <typename T>
__global__ __launch_bounds__(LEAF_THREADS) void k_leaf_spec(int64_t Np, int64_t c0, T *__restrict__ A,
                                                            int64_t lda, T *__restrict__ LT, int64_t k0,
                                                            int nrt, int nct, T *__restrict__ DG,
                                                            const T *__restrict__ DGprev, int64_t cprev,
                                                            int *__restrict__ flags)
{
    leaf_body<T>(blockIdx.x, Np, c0, A, lda, LT, NB_OUT, c0 - k0, nrt, nct, DG, DGprev, cprev, flags);
}

// copy a 64x64 diagonal block from DG into A (the last leaf's block)
template <typename T>
__global__ __launch_bounds__(256) void k_put_diag(int64_t c0, T *__restrict__ A, int64_t lda,
                                                  const T *__restrict__ DG, const int *flags)
{
    if (ld_flag(&flags[FLAG_FAIL])) return;
    for (int e = threadIdx.x; e < NB_LEAF * NB_LEAF; e += 256) {
        const int i = e % NB_LEAF, j = e / NB_LEAF;
        A[(c0 + i) + (c0 + j) * lda] = DG[i + j * NB_LEAF];
    }
}

// The FP16/BF16 Schur tile (gemm16_tile) and its XCD-aware tile order are in n3p_gemm.hpp.

template <typename T, int TM, int TN, int WGM, int WGN, int KC>
__global__ __launch_bounds__(WGM *WGN * 64) void k_gemm16(int M, int N, int K,
                                                          const T *__restrict__ At, int64_t ldat,
                                                          const T *__restrict__ B, int64_t ldb,
                                                          T *__restrict__ C, int64_t ldc,
                                                          int *__restrict__ flags, int check_abort)
{
    if (check_abort && block_flag(&flags[FLAG_FAIL])) return;
    const int ntm = M / TM, ntn = N / TN;
    int tm, tn;
    grouped_tile(xcd_tile(blockIdx.x, ntm * ntn), ntm, ntn, tm, tn);
    __shared__ __attribute__((aligned(16))) T lds[gemm16_lds_elems<TM, TN, KC>()];
    gemm16_tile<T, TM, TN, WGM, WGN, KC>(tm * TM, tn * TN, K, At, ldat, B, ldb, C, ldc, flags, lds);
}

// Two independent updates with the same K in one launch (tiles of the first,
// then of the second): after a leaf, the rest of its panel (below) and the
// row block right of the panel write disjoint parts of C and only read L and U.
struct GemmProb {
    int M, N;
    const void *At;
    int64_t ldat;
    const void *B;
    int64_t ldb;
    void *C;
    int64_t ldc;
};

// ========================================== Schur GEMM, FP32/FP64 matrix cores
// C -= At^T B for one or two problems with the same K (the two updates that
// follow a panel are independent).  64x64 block tile, 4 waves of 32x32 (2x2
// fragments of 16x16); K in chunks of 32 through two LDS buffers, the chunk
// after next in registers.  A K = 64 launch is one memory round trip: its
// operands, C and the flag are requested together; the LDS rows keep K
// contiguous, padded by two (FP32: four) elements, so 16-byte stores and the
// fragments' reads (16 rows x 4 k) are free of bank conflicts.  The fragments
// are computed transposed (the A rows as the second operand), so a wave's C
// accesses are runs of 16 rows.
// Small launches are bound by that round trip, large ones by the matrix cores
// (50 TFLOP/s at M = N = 1984, K = 1024).
// Measured, FP64: one tile, K = 64: 10.3 -> 6.0 us; 225 tiles, K = 1024: 81 ->
// 51 us; 961 tiles: 198 -> 162 us (from 16-wide chunks read without looking
// ahead and stored element by element); the updates of n = 3000: 1460 -> 670 us
// in half the launches.
template <typename T>
__global__ __launch_bounds__(256) void k_gemm_mfma4(GemmProb p1, GemmProb p2, int K,
                                                    int *__restrict__ flags, int check_abort)
{
    typedef typename mfma16x4<T>::acc_t acc_t;
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    constexpr int TM = 64, KC = 32, CH = 16 / (int)sizeof(T), CPR = KC / CH;
    constexpr int KP = KC + CH, NL = TM * CPR / 256;  // 16-byte chunks a thread and operand
    __shared__ __attribute__((aligned(16))) T As[2][TM * KP];
    __shared__ __attribute__((aligned(16))) T Bs[2][TM * KP];
    __shared__ int s_flag;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int fl = 0;
    if (check_abort && tid == 0) fl = ld_flag(&flags[FLAG_FAIL]);
    const int n1 = (p1.M / TM) * (p1.N / TM), n2 = (p2.M / TM) * (p2.N / TM);
    int tile = xcd_tile(blockIdx.x, n1 + n2), tm, tn;
    const bool second = tile >= n1;
    const GemmProb &p = second ? p2 : p1;
    grouped_tile(second ? tile - n1 : tile, p.M / TM, p.N / TM, tm, tn);
    const T *At = (const T *)p.At + (int64_t)(tm * TM) * p.ldat;
    const T *B = (const T *)p.B + (int64_t)(tn * TM) * p.ldb;
    const int64_t ldat = p.ldat, ldb = p.ldb;
    u32x4 ra[2][NL], rb[2][NL];
    auto load = [&](u32x4 (&xa)[NL], u32x4 (&xb)[NL], int kk) {
#pragma unroll
        for (int c = 0; c < NL; ++c) {
            const int ch = tid + c * 256, r = ch / CPR, seg = (ch % CPR) * CH;
            xa[c] = *(const u32x4 *)(At + r * ldat + kk + seg);
            xb[c] = *(const u32x4 *)(B + r * ldb + kk + seg);
        }
    };
    auto stage = [&](int buf, const u32x4 (&xa)[NL], const u32x4 (&xb)[NL]) {
#pragma unroll
        for (int c = 0; c < NL; ++c) {
            const int ch = tid + c * 256, r = ch / CPR, seg = (ch % CPR) * CH;
            *(u32x4 *)&As[buf][r * KP + seg] = xa[c];
            *(u32x4 *)&Bs[buf][r * KP + seg] = xb[c];
        }
    };
    load(ra[0], rb[0], 0);
    load(ra[1], rb[1], KC);
    const int wm = (wave & 1) * 32, wn = (wave >> 1) * 32, ci = lane & 15, kl = lane >> 4;
    T *C = (T *)p.C + (int64_t)(tn * TM + wn) * p.ldc + tm * TM + wm + ci;
    const int64_t ldc = p.ldc;
    acc_t cv[2][2], acc[2][2];
#pragma unroll
    for (int fm = 0; fm < 2; ++fm)
#pragma unroll
        for (int fn = 0; fn < 2; ++fn)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                cv[fm][fn][q] = C[(fn * 16 + mfma16x4<T>::row(lane, q)) * ldc + fm * 16];
                acc[fm][fn][q] = 0;
            }
    auto product = [&](int buf) {
#pragma unroll
        for (int ks = 0; ks < KC; ks += 4) {
            T a[2], b[2];
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                a[f] = As[buf][(wm + f * 16 + ci) * KP + ks + kl];
                b[f] = Bs[buf][(wn + f * 16 + ci) * KP + ks + kl];
            }
#pragma unroll
            for (int fm = 0; fm < 2; ++fm)
#pragma unroll
                for (int fn = 0; fn < 2; ++fn)
                    acc[fm][fn] = mfma16x4<T>::op(b[fn], a[fm], acc[fm][fn]);
        }
    };
    stage(0, ra[0], rb[0]);
    if (tid == 0) s_flag = fl;
    __syncthreads();
    if (s_flag) return;  // block-uniform
    for (int kk = 0; kk < K; kk += 2 * KC) {
        const bool more = kk + 2 * KC < K;
        if (more) load(ra[0], rb[0], kk + 2 * KC);
        product(0);
        stage(1, ra[1], rb[1]);
        __syncthreads();
        if (more) load(ra[1], rb[1], kk + 3 * KC);
        product(1);
        if (more) {
            stage(0, ra[0], rb[0]);
            __syncthreads();
        }
    }
    bool bad = false;
#pragma unroll
    for (int fm = 0; fm < 2; ++fm)
#pragma unroll
        for (int fn = 0; fn < 2; ++fn)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const T v = cv[fm][fn][q] - acc[fm][fn][q];
                bad |= !isfinite((double)v);
                C[(fn * 16 + mfma16x4<T>::row(lane, q)) * ldc + fm * 16] = v;
            }
    if (bad) set_flag(&flags[FLAG_NONFINITE], 1);
}

template <typename T>
__global__ __launch_bounds__(256) void k_check_finite(int64_t Np, const T *__restrict__ A,
                                                      int64_t lda, int *__restrict__ flags)
{
    const int64_t j = blockIdx.x;
    bool bad = false;
    for (int64_t i = threadIdx.x; i < Np; i += 256) bad |= !isfinite((double)to_f32(A[i + j * lda]));
    if (bad) set_flag(&flags[FLAG_NONFINITE], 1);
}

// ================================================================ launchers
template <typename T>
static hipError_t leaf_spec_t(int64_t Np, int64_t c0, void *A, int64_t lda, void *LT, int64_t k0,
                              void *DG, const void *DGprev, int64_t cprev, int *flags,
                              hipStream_t s)
{
    const int64_t below = Np - c0 - NB_LEAF;  // a multiple of NB_LEAF
    const int nrt = (int)(below / NB_LEAF);
    const int nct = nrt;
    const unsigned grid = (unsigned)std::max(1, nrt + nct);
    hipLaunchKernelGGL(k_leaf_spec<T>, dim3(grid), dim3(LEAF_THREADS), 0, s, Np, c0, (T *)A, lda,
                       (T *)LT, k0, nrt, nct, (T *)DG, (const T *)DGprev, cprev, flags);
    return hipGetLastError();
}

hipError_t launch_leaf_spec2(int prec, int64_t Np, int64_t c0, void *A, int64_t lda, void *LT,
                             int64_t k0, void *DG, const void *DGprev, int64_t cprev, int *flags,
                             hipStream_t s)
{
    switch (prec) {
    case N3P_FP32: return leaf_spec_t<float>(Np, c0, A, lda, LT, k0, DG, DGprev, cprev, flags, s);
    case N3P_FP64: return leaf_spec_t<double>(Np, c0, A, lda, LT, k0, DG, DGprev, cprev, flags, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_put_diag(int prec, int64_t c0, void *A, int64_t lda, const void *DG,
                           const int *flags, hipStream_t s)
{
    switch (prec) {
    case N3P_FP16: hipLaunchKernelGGL(k_put_diag<f16>, dim3(1), dim3(256), 0, s, c0, (f16 *)A, lda, (const f16 *)DG, flags); break;
    case N3P_BF16: hipLaunchKernelGGL(k_put_diag<bf16>, dim3(1), dim3(256), 0, s, c0, (bf16 *)A, lda, (const bf16 *)DG, flags); break;
    case N3P_FP32: hipLaunchKernelGGL(k_put_diag<float>, dim3(1), dim3(256), 0, s, c0, (float *)A, lda, (const float *)DG, flags); break;
    case N3P_FP64: hipLaunchKernelGGL(k_put_diag<double>, dim3(1), dim3(256), 0, s, c0, (double *)A, lda, (const double *)DG, flags); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <typename T, int TM, int TN, int WGM, int WGN, int KC>
static void gemm16_go(int64_t M, int64_t N, int64_t K, const void *At, int64_t ldat, const void *B,
                      int64_t ldb, void *C, int64_t ldc, int *flags, bool ca, hipStream_t s)
{
    const unsigned grid = (unsigned)((M / TM) * (N / TN));
    hipLaunchKernelGGL((k_gemm16<T, TM, TN, WGM, WGN, KC>), dim3(grid), dim3(WGM * WGN * 64), 0, s,
                       (int)M, (int)N, (int)K, (const T *)At, ldat, (const T *)B, ldb, (T *)C, ldc,
                       flags, (int)ca);
}

template <typename T>
static hipError_t gemm16_t(int64_t M, int64_t N, int64_t K, const void *At, int64_t ldat,
                           const void *B, int64_t ldb, void *C, int64_t ldc, int *flags, bool ca,
                           hipStream_t s)
{
    if (M % 64 || N % 64 || K % 64) return hipErrorInvalidValue;
    if (M % 256 == 0 && N % 256 == 0 && M * N >= (int64_t)256 * 256 * 128)
        gemm16_go<T, 256, 256, 2, 4, 32>(M, N, K, At, ldat, B, ldb, C, ldc, flags, ca, s);
    else if (M % 128 == 0 && N % 128 == 0 && M * N >= (int64_t)128 * 128 * 128)
        gemm16_go<T, 128, 128, 2, 2, 32>(M, N, K, At, ldat, B, ldb, C, ldc, flags, ca, s);
    else
        gemm16_go<T, 64, 64, 2, 2, 32>(M, N, K, At, ldat, B, ldb, C, ldc, flags, ca, s);
    return hipGetLastError();
}

template <typename T>
static hipError_t gemm4_pair_t(GemmProb a, GemmProb b, int K, int *flags, bool ca, hipStream_t s)
{
    const unsigned g = (unsigned)((a.M / 64) * (a.N / 64) + (b.M / 64) * (b.N / 64));
    hipLaunchKernelGGL(k_gemm_mfma4<T>, dim3(g), dim3(256), 0, s, a, b, K, flags, (int)ca);
    return hipGetLastError();
}

template <typename T>
static hipError_t gemm4_t(int64_t M, int64_t N, int64_t K, const void *At, int64_t ldat,
                          const void *B, int64_t ldb, void *C, int64_t ldc, int *flags, bool ca,
                          hipStream_t s)
{
    if (M % 64 || N % 64 || K % 64) return hipErrorInvalidValue;
    const GemmProb a{(int)M, (int)N, At, ldat, B, ldb, C, ldc};
    GemmProb none = a;
    none.M = 0;
    return gemm4_pair_t<T>(a, none, (int)K, flags, ca, s);
}

hipError_t launch_gemm_sub(int prec, int64_t M, int64_t N, int64_t K, const void *At, int64_t ldat,
                           const void *B, int64_t ldb, void *C, int64_t ldc, int *flags,
                           bool check_abort, hipStream_t s)
{
    if (M <= 0 || N <= 0 || K <= 0) return hipSuccess;
    switch (prec) {
    case N3P_FP16: return gemm16_t<f16>(M, N, K, At, ldat, B, ldb, C, ldc, flags, check_abort, s);
    case N3P_BF16: return gemm16_t<bf16>(M, N, K, At, ldat, B, ldb, C, ldc, flags, check_abort, s);
    case N3P_FP32: return gemm4_t<float>(M, N, K, At, ldat, B, ldb, C, ldc, flags, check_abort, s);
    case N3P_FP64: return gemm4_t<double>(M, N, K, At, ldat, B, ldb, C, ldc, flags, check_abort, s);
    }
    return hipErrorInvalidValue;
}

// C1 -= At1^T B1 and C2 -= At2^T B2 (same K) in one launch; FP32/FP64 only,
// every M, N, K a multiple of 64.  An empty problem is allowed.
hipError_t launch_gemm_pair(int prec, int64_t M1, int64_t N1, const void *At1, int64_t ldat1,
                            const void *B1, int64_t ldb1, void *C1, int64_t ldc1, int64_t M2,
                            int64_t N2, const void *At2, int64_t ldat2, const void *B2,
                            int64_t ldb2, void *C2, int64_t ldc2, int64_t K, int *flags,
                            hipStream_t s)
{
    if (M1 % 64 || N1 % 64 || M2 % 64 || N2 % 64 || K % 64 || K <= 0) return hipErrorInvalidValue;
    GemmProb a{(int)M1, (int)N1, At1, ldat1, B1, ldb1, C1, ldc1};
    GemmProb b{(int)M2, (int)N2, At2, ldat2, B2, ldb2, C2, ldc2};
    if (M1 <= 0 || N1 <= 0) { a.M = 0; a.N = 64; }
    if (M2 <= 0 || N2 <= 0) { b.M = 0; b.N = 64; }
    if (a.M == 0 && b.M == 0) return hipSuccess;
    switch (prec) {
    case N3P_FP32: return gemm4_pair_t<float>(a, b, (int)K, flags, true, s);
    case N3P_FP64: return gemm4_pair_t<double>(a, b, (int)K, flags, true, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_check_factor_finite(int prec, int64_t Np, const void *A, int64_t lda, int *flags,
                                      hipStream_t s)
{
    switch (prec) {
    case N3P_FP16: hipLaunchKernelGGL(k_check_finite<f16>, dim3((unsigned)Np), dim3(256), 0, s, Np, (const f16 *)A, lda, flags); break;
    case N3P_BF16: hipLaunchKernelGGL(k_check_finite<bf16>, dim3((unsigned)Np), dim3(256), 0, s, Np, (const bf16 *)A, lda, flags); break;
    case N3P_FP32: hipLaunchKernelGGL(k_check_finite<float>, dim3((unsigned)Np), dim3(256), 0, s, Np, (const float *)A, lda, flags); break;
    case N3P_FP64: hipLaunchKernelGGL(k_check_finite<double>, dim3((unsigned)Np), dim3(256), 0, s, Np, (const double *)A, lda, flags); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}


// ====================================================== batched engine kernels
// Leaf `leaf` (columns 64 leaf .. +64) of every slot that factors this step:
// the same leaf body as the single factorisation, with L21 kept transposed in
// the slot's LT (ld 64) for the rank-64 update that follows.  A slot's last
// leaf has no tiles and writes its diagonal block straight into A.
template <typename T>
__global__ __launch_bounds__(LEAF_THREADS) void k_b_leaf(const BDesc *__restrict__ d,
                                                         const BState *__restrict__ st, int nslots,
                                                         int leaf)
{
    __shared__ int off[B_MAX_SLOTS + 1];
    const int64_t c0 = (int64_t)leaf * NB_LEAF;
    const int total = b_offsets(nslots, off, [&](int s) {
        const int nl = b_factor_leaves(d[s], st[s]) - leaf;
        return nl > 1 ? 2 * (nl - 1) : std::max(nl, 0);
    });
    for (int item = blockIdx.x; item < total; item += gridDim.x) {
        const int s = b_find(off, nslots, item);
        const BDesc &q = d[s];
        const int nrt = (int)((q.Np - c0 - NB_LEAF) / NB_LEAF);
        T *DGs = (T *)q.DG;
        T *DG = nrt > 0 ? DGs + (leaf % 2) * NB_LEAF * NB_LEAF : nullptr;
        const T *DGprev = leaf > 0 ? DGs + ((leaf - 1) % 2) * NB_LEAF * NB_LEAF : nullptr;
        leaf_body<T>(item - off[s], q.Np, c0, (T *)q.A, q.Np, (T *)q.LT, NB_LEAF, 0, nrt, nrt, DG,
                     DGprev, c0 - NB_LEAF, q.flags);
        __syncthreads();
    }
}

// Rank-64 Schur update after leaf `leaf`: A22 -= L21 U12 for every slot that
// factors this step, in TM x TM tiles (TM = 64: every trailing size is a
// multiple of 64).
template <typename T, int KC>
__global__ __launch_bounds__(256) void k_b_gemm(const BDesc *__restrict__ d,
                                                const BState *__restrict__ st, int nslots, int leaf)
{
    constexpr int TM = 64;
    __shared__ int off[B_MAX_SLOTS + 1];
    __shared__ __attribute__((aligned(16))) T lds[gemm16_lds_elems<TM, TM, KC>()];
    const int64_t c0 = (int64_t)leaf * NB_LEAF, c1 = c0 + NB_LEAF;
    const int total = b_offsets(nslots, off, [&](int s) {
        const int m = std::max(b_factor_leaves(d[s], st[s]) - leaf - 1, 0);
        return m * m;
    });
    for (int item = blockIdx.x; item < total; item += gridDim.x) {
        const int s = b_find(off, nslots, item);
        const BDesc &q = d[s];
        if (ld_flag(&q.flags[FLAG_FAIL])) continue;  // abandoned: needs interchanges
        const int m = (int)((q.Np - c1) / TM), local = item - off[s];
        const int tm = local % m, tn = local / m;
        T *A = (T *)q.A;
        const int64_t Np = q.Np;
        gemm16_tile<T, TM, TM, 2, 2, KC>(tm * TM, tn * TM, NB_LEAF, (const T *)q.LT + c1 * NB_LEAF,
                                         NB_LEAF, A + c0 + c1 * Np, Np, A + c1 + c1 * Np, Np,
                                         q.flags, lds);
        __syncthreads();
    }
}

hipError_t launch_b_leaf(int prec, const BDesc *d, const BState *st, int nslots, int leaf,
                         int grid, hipStream_t s)
{
    switch (prec) {
    case N3P_FP16: hipLaunchKernelGGL(k_b_leaf<f16>, dim3(grid), dim3(LEAF_THREADS), 0, s, d, st, nslots, leaf); break;
    case N3P_BF16: hipLaunchKernelGGL(k_b_leaf<bf16>, dim3(grid), dim3(LEAF_THREADS), 0, s, d, st, nslots, leaf); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_b_gemm(int prec, const BDesc *d, const BState *st, int nslots, int leaf,
                         int kc, int grid, hipStream_t s)
{
    if (prec == N3P_FP16) {
        if (kc == 64) hipLaunchKernelGGL((k_b_gemm<f16, 64>), dim3(grid), dim3(256), 0, s, d, st, nslots, leaf);
        else hipLaunchKernelGGL((k_b_gemm<f16, 32>), dim3(grid), dim3(256), 0, s, d, st, nslots, leaf);
    } else if (prec == N3P_BF16) {
        if (kc == 64) hipLaunchKernelGGL((k_b_gemm<bf16, 64>), dim3(grid), dim3(256), 0, s, d, st, nslots, leaf);
        else hipLaunchKernelGGL((k_b_gemm<bf16, 32>), dim3(grid), dim3(256), 0, s, d, st, nslots, leaf);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace n3p
