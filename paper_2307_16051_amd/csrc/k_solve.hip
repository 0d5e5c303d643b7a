// k_solve.hip -- the preconditioner-vector product U^{-1} L^{-1} P r
// (Section 2.2) and the single-precision residual r = b - A u.
//
// Triangular solves: one persistent launch per solve.  Row blocks of BS rows
// are taken in dependency order through an atomic ticket (a block only waits
// on blocks with smaller tickets, which are already running, so the waits
// always end).  Block i inverts its diagonal block and premultiplies the
// tile of its nearest predecessor by that inverse while the chain is still
// far away, accumulates the contributions of the other finished blocks as
// they are published, and once its nearest predecessor publishes, finishes
// with one BS x BS product and publishes its piece of the solution as words
// stamped with the launch's epoch (no flag reset between launches).  Factors are read in their
// storage precision and promoted in registers (interprecision transfer on
// the fly, Section 2.3).  Every wait is bounded; an expired wait raises
// FLAG_TIMEOUT and the block proceeds so that the grid always drains.
#include <algorithm>
#include <mutex>

#include "n3p_internal.hpp"

namespace n3p {

constexpr int SPIN_LIMIT = 1 << 24;

// Solution values are published as 64-bit words (epoch << 32 | 32 bits of
// data): FP32 values take one word, FP64 values two.  A reader polls the words
// it needs until their tag equals the launch's epoch, so the value arrives in
// the same memory round trip as its readiness (no separate flag), and no
// cache-wide fence is needed: the words are written and read with
// agent-scope (coherent) atomic accesses.
template <typename V> struct tagged;
template <> struct tagged<float> {
    static constexpr int W = 1;
    static __device__ __forceinline__ void put(uint64_t *t, int64_t i, float v, uint32_t ep)
    {
        const uint64_t w = ((uint64_t)ep << 32) | (uint32_t)__float_as_uint(v);
        __hip_atomic_store(&t[i], w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
};
template <> struct tagged<double> {
    static constexpr int W = 2;
    static __device__ __forceinline__ void put(uint64_t *t, int64_t i, double v, uint32_t ep)
    {
        const uint64_t b = (uint64_t)__double_as_longlong(v);
        __hip_atomic_store(&t[2 * i], ((uint64_t)ep << 32) | (b & 0xffffffffULL), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&t[2 * i + 1], ((uint64_t)ep << 32) | (b >> 32), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
};

// sync layout: int ticket at [0]; tagged words (uint64) from byte offset 16
__device__ __forceinline__ uint64_t *tag_words(int *sync) { return (uint64_t *)(sync + 4); }

// The next block of this launch in dependency order, 0 .. nblocks - 1.  The
// counter is never reset: the caller clears it once, launches with epochs
// 1, 2, ... and the same number of blocks each time, so this launch's tickets
// start at (epoch - 1) nblocks (a launch of its own to clear it took 3 us).
__device__ __forceinline__ int take_ticket(int *sync, uint32_t epoch, uint32_t nblocks)
{
    const uint32_t t = (uint32_t)__hip_atomic_fetch_add(&sync[0], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return (int)(t - (epoch - 1) * nblocks);
}

// One published value per lane: lane c of a wavefront fetches the word(s) of
// column c of a tile, re-polls until every lane's tag matches, and then the
// values are broadcast lane by lane (v_readlane) into the row updates.
template <typename V>
struct lane_word {
    uint64_t w[tagged<V>::W];
    __device__ __forceinline__ void issue(const uint64_t *t, int64_t idx, bool valid)
    {
#pragma unroll
        for (int h = 0; h < tagged<V>::W; ++h)
            w[h] = valid ? __hip_atomic_load(&t[idx * tagged<V>::W + h], __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT)
                         : 0;
    }
    // backoff: extra sleep between polls, in units of 256 cycles.  A block
    // waiting for a tile far behind its own row block has time to spare, and
    // every poll of the newest words competes with the poll of the block
    // that needs them next, so far blocks poll rarely.
    __device__ __forceinline__ void settle(const uint64_t *t, int64_t idx, bool valid, uint32_t ep,
                                           int *spins, int *flags, int backoff = 0)
    {
        for (;;) {
            if (ready(valid, ep)) return;
            __builtin_amdgcn_s_sleep(1);
            for (int k = 0; k < backoff; ++k) __builtin_amdgcn_s_sleep(4);
            *spins += backoff > 0 ? backoff : 0;  // the bound counts sleeps, not polls
            if (++*spins > SPIN_LIMIT) {
                set_flag(&flags[FLAG_TIMEOUT], 1);
                return;
            }
            bool ok = true;
            if (valid) {
#pragma unroll
                for (int h = 0; h < tagged<V>::W; ++h) ok &= (uint32_t)(w[h] >> 32) == ep;
            }
            if (!ok) issue(t, idx, valid);
        }
    }
    __device__ __forceinline__ bool ready(bool valid, uint32_t ep) const
    {
        bool ok = true;
        if (valid) {
#pragma unroll
            for (int h = 0; h < tagged<V>::W; ++h) ok &= (uint32_t)(w[h] >> 32) == ep;
        }
        return __all(ok);
    }
    // The wait on the last hand-off before a block can finish.  settle()
    // re-polls only after its previous poll has returned, so a value that
    // lands just after a poll passed is seen almost two memory round trips
    // later.  Here, once the first poll (*this, already issued) has missed,
    // four polls are kept in flight, issued a quarter of a round trip apart:
    // the value is seen about one trip after it lands.  Straight-line code (fully
    // unrolled), so each check waits for its own poll only; after RING
    // rounds it falls back to settle().
    template <int RING>
    __device__ __forceinline__ void settle_ring(const uint64_t *t, int64_t idx, bool valid,
                                                uint32_t ep, int *spins, int *flags)
    {
        if (ready(valid, ep)) return;
        issue(t, idx, valid);
        lane_word b, c, d;
        __builtin_amdgcn_s_sleep(9);
        b.issue(t, idx, valid);
        __builtin_amdgcn_s_sleep(9);
        c.issue(t, idx, valid);
        __builtin_amdgcn_s_sleep(9);
        d.issue(t, idx, valid);
#pragma unroll
        for (int r = 0; r < RING; ++r) {
            if (ready(valid, ep)) return;
            issue(t, idx, valid);
            if (b.ready(valid, ep)) { *this = b; return; }
            b.issue(t, idx, valid);
            if (c.ready(valid, ep)) { *this = c; return; }
            c.issue(t, idx, valid);
            if (d.ready(valid, ep)) { *this = d; return; }
            d.issue(t, idx, valid);
        }
        *spins += 4 * RING;
        settle(t, idx, valid, ep, spins, flags);
    }
    __device__ __forceinline__ V value() const
    {
        if constexpr (tagged<V>::W == 1) {
            return __uint_as_float((uint32_t)w[0]);
        } else {
            const uint64_t lo = (uint32_t)w[0], hi = (uint32_t)w[1];
            return __longlong_as_double((long long)((hi << 32) | lo));
        }
    }
};

template <typename T, typename V, int BS>
__device__ __forceinline__ void load_tile_row(V (&fv)[BS], const T *__restrict__ LU, int64_t lda,
                                              int64_t rowc, int64_t c0, int64_t n)
{
    // unconditional loads (column index clamped in bounds) so that all BS
    // loads issue back to back; entries past column n-1 are zeroed after
    T raw[BS];
#pragma unroll
    for (int c = 0; c < BS; ++c) raw[c] = LU[rowc + std::min<int64_t>(c0 + c, n - 1) * lda];
#pragma unroll
    for (int c = 0; c < BS; ++c) fv[c] = c0 + c < n ? (V)to_f32(raw[c]) : (V)0;
}

// Diagonal-block helpers.  Each block inverts its own BS x BS diagonal block
// D (row-major in Dr) and forms Mx = D^{-1} E, with E the neighbouring
// off-diagonal tile it depends on last (in Eb).  Then only one product with
// the neighbour's solution is left after it arrives:
// lower x_b = D^{-1} (b_b - sum_{j<b-1} L_bj x_j) - D^{-1} L_{b,b-1} x_{b-1},
// upper x_b = D^{-1} (y_b - sum_{j>b+1} U_bj x_j) - D^{-1} U_{b,b+1} x_{b+1}.
// (Rounding differs from substitution only in the order of the sums.)
//
// This prologue is what a solve of few blocks waits for: the first block
// cannot publish before it, and at n = 256 it was 15 of 24 us (the tiles
// fetched one load at a time, and 64 rows substituted by one wavefront).  So
// all 32 loads of a thread go out together, and the inverse is built by
// blocks on all four wavefronts: four 16 x 16 inverses by substitution, then
// 16 -> 32 -> 64 by X = -D_aa^{-1} (D_ab D_bb^{-1}) on the FP32 / FP64 matrix
// cores, which also form Mx: about 14 us less per solve (n = 1000, 42 solves:
// 6.00 -> 5.40 ms; n = 6001 FP16: 374 -> 307 us for the pair).  All LDS matrices have row stride LS (odd: a
// column's accesses fall into different banks).
template <int BS> struct lds_stride { static constexpr int LS = BS + 1; };

// one 16 x 16 fragment of P Q, K deep: P at Pm (row stride LS), Q at Qm
template <typename V, int K, int LS>
__device__ __forceinline__ typename mfma16x4<V>::acc_t frag_mul(const V *__restrict__ Pm,
                                                                const V *__restrict__ Qm, int lane)
{
    const int r = lane & 15, g = lane >> 4;
    typename mfma16x4<V>::acc_t acc = {0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < K; k += 4)
        acc = mfma16x4<V>::op(Pm[r * LS + k + g], Qm[(k + g) * LS + r], acc);
    return acc;
}
// acc -= P T with T a fragment as an earlier product left it: register q of
// lane l holds row row(l, q) of T, so step q takes that k in both operands
template <typename V, int LS>
__device__ __forceinline__ void frag_sub(typename mfma16x4<V>::acc_t &acc, const V *__restrict__ Pm,
                                         const typename mfma16x4<V>::acc_t &t, int lane)
{
#pragma unroll
    for (int q = 0; q < 4; ++q)
        acc = mfma16x4<V>::op(-Pm[(lane & 15) * LS + mfma16x4<V>::row(lane, q)], t[q], acc);
}
template <typename V, int LS>
__device__ __forceinline__ void frag_store(V *__restrict__ X, const typename mfma16x4<V>::acc_t &a,
                                           int lane)
{
#pragma unroll
    for (int q = 0; q < 4; ++q) X[mfma16x4<V>::row(lane, q) * LS + (lane & 15)] = a[q];
}

// Di = D^{-1} (LOWER: unit lower; else upper with reciprocals rd of its
// diagonal), then Dr = Di Eb if `mx`.  All 256 threads; Di zeroed and Dr
// (zero on and beyond the diagonal's wrong side) and Eb stored by the caller,
// without a barrier since.  Ends without a barrier.
template <typename V, int BS, bool LOWER>
__device__ __forceinline__ void diag_inverse_mx(V *__restrict__ Dr, const V *__restrict__ rd,
                                                const V *__restrict__ Eb, V *__restrict__ Di,
                                                bool mx, int lane, int wv)
{
    static_assert(BS == 64, "four wavefronts, one 16-row block each");
    constexpr int LS = lds_stride<BS>::LS;
    typedef typename mfma16x4<V>::acc_t acc_t;
    __syncthreads();
    {  // 16 x 16 blocks, lane & 15 = column of the inverse
        const V *D = Dr + 16 * wv * (LS + 1);
        const int c = lane & 15;
        V xi[16];
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            const int i = LOWER ? s : 15 - s;
            V a[2] = {c == i ? (V)1 : (V)0, 0};
#pragma unroll
            for (int u = 0; u < s; ++u) {
                const int k = LOWER ? u : 15 - u;
                a[u & 1] -= D[i * LS + k] * xi[k];
            }
            xi[i] = a[0] + a[1];
            if constexpr (!LOWER) xi[i] *= rd[16 * wv + i];
        }
        if (lane < 16) {
#pragma unroll
            for (int i = 0; i < 16; ++i) Di[(16 * wv + i) * LS + 16 * wv + c] = xi[i];
        }
    }
    __syncthreads();
    constexpr int A = LOWER ? 1 : 0, B = 1 - A;  // row and column half of the coupling block
    if (wv < 2) {                                // 16 -> 32, one pair of blocks per wavefront
        const int ra = 32 * wv + 16 * A, cb = 32 * wv + 16 * B;
        const acc_t t = frag_mul<V, 16, LS>(Dr + ra * LS + cb, Di + cb * LS + cb, lane);
        acc_t x = {0, 0, 0, 0};
        frag_sub<V, LS>(x, Di + ra * LS + ra, t, lane);
        frag_store<V, LS>(Di + ra * LS + cb, x, lane);
    }
    __syncthreads();
    {  // 32 -> 64, one 16 x 16 fragment of the coupling block per wavefront
        const int ra = 32 * A, cb = 32 * B, i = wv >> 1, j = wv & 1;
        acc_t x = {0, 0, 0, 0};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const acc_t t = frag_mul<V, 32, LS>(Dr + (ra + 16 * h) * LS + cb,
                                                Di + cb * LS + cb + 16 * j, lane);
            frag_sub<V, LS>(x, Di + (ra + 16 * i) * LS + ra + 16 * h, t, lane);
        }
        frag_store<V, LS>(Di + (ra + 16 * i) * LS + cb + 16 * j, x, lane);
    }
    __syncthreads();
    if (!mx) return;
    // Mx: 16 columns per wavefront; the inverse's zero 16 x 16 blocks left out
    const int r = lane & 15, g = lane >> 4;
    V e[BS / 4];
#pragma unroll
    for (int s = 0; s < BS / 4; ++s) e[s] = Eb[(4 * s + g) * LS + 16 * wv + r];
#pragma unroll
    for (int i = 0; i < BS / 16; ++i) {
        acc_t m = {0, 0, 0, 0};
#pragma unroll
        for (int s = LOWER ? 0 : 4 * i; s < (LOWER ? 4 * (i + 1) : BS / 4); ++s)
            m = mfma16x4<V>::op(Di[(16 * i + r) * LS + 4 * s + g], e[s], m);
        frag_store<V, LS>(Dr + 16 * i * LS + 16 * wv, m, lane);
    }
}

// sum_c r[c] v[c] with v held one value per lane and passed through LDS (vb:
// this wavefront's BS entries), four independent partial sums: one store and
// BS/4 broadcast reads instead of BS readlanes, which the compiler chains
// through one SGPR with a wait state each.  vb must be 16-byte aligned.
template <typename V, int BS>
__device__ __forceinline__ V row_times_lds(const V (&r)[BS], V v, V *vb, int lane)
{
    constexpr int K = 16 / sizeof(V);
    vb[lane] = v;  // one wavefront's LDS accesses complete in order
    V a[4] = {0, 0, 0, 0};
#pragma unroll
    for (int c = 0; c < BS; c += K) {
        V u[K];
        __builtin_memcpy(u, vb + c, 16);
#pragma unroll
        for (int k = 0; k < K; ++k) a[(c + k) & 3] += r[c + k] * u[k];
    }
    return (a[0] + a[1]) + (a[2] + a[3]);
}
// row `lane` of an LDS matrix with stride BS + 1, into registers
template <typename V, int BS>
__device__ __forceinline__ void load_row(V (&r)[BS], const V *__restrict__ R, int lane)
{
#pragma unroll
    for (int c = 0; c < BS; ++c) r[c] = R[lane * (BS + 1) + c];
}

// ------------------------------------------------------- one row block
// round_out (both solves): every solution entry is rounded to the factor
// type T as it is formed, before later blocks use it -- the solve held in
// the low precision for the scaled correction of eq. (2.19) (Section 2.3).
//
// Block `blk` owns rows [blk*BS, blk*BS + BS) (lane = row).  rhs(row) is the
// right-hand side of a row, out(row, w) takes its solution; both are called
// by wavefront 0 for rows < n.
template <typename V, int BS> struct TrsvLds {
    static constexpr int LS = lds_stride<BS>::LS;
    V Dr[BS * LS];  // D, then Mx
    V Eb[BS * LS];  // L_{b,b-1} or U_{b,b+1}
    V Di[BS * LS];  // D^{-1}
    V rd[BS];
    V part[4][BS];
    __attribute__((aligned(16))) V vb[4][BS];  // each wavefront's broadcast vector
};

// Lower: wavefront w consumes tiles w, w+4, ... below blk - 1, keeping the
// next tile's loads in flight while it consumes the current one.  Tile
// blk - 1 enters through Mx = D^{-1} L_{b,b-1}.
template <typename T, typename V, int BS, typename Rhs, typename Out>
__device__ __forceinline__ void trsv_lower_block(TrsvLds<V, BS> &sh, int blk, int64_t n,
                                                 const T *__restrict__ LU, int64_t lda,
                                                 uint64_t *tags, uint32_t epoch,
                                                 int *__restrict__ flags, int round_out, Rhs rhs,
                                                 Out out)
{
    static_assert(BS == 64, "a wavefront spans one tile");
    constexpr int LS = TrsvLds<V, BS>::LS, PT = BS / 4;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t r0 = (int64_t)blk * BS;
    const int64_t row = r0 + lane;
    const bool rv = row < n;
    const int64_t rowc = rv ? row : 0;
    V acc = 0;
    int spins = 0;
    V fv[BS], fvn[BS];
    lane_word<V> cur, nxt;
    const int last = blk - 1;  // tiles jb < last go through the loop
    {
        // lane = row, columns wv, wv + 4, ...: all loads first (columns
        // clamped in bounds), then the zeros and the stores to LDS
        T d[PT], e[PT];
#pragma unroll
        for (int k = 0; k < PT; ++k)
            d[k] = LU[rowc + std::min<int64_t>(r0 + wv + 4 * k, n - 1) * lda];
        if (blk > 0) {
#pragma unroll
            for (int k = 0; k < PT; ++k) e[k] = LU[rowc + (r0 - BS + wv + 4 * k) * lda];
        }
#pragma unroll
        for (int k = 0; k < PT; ++k) {
            const int j = wv + 4 * k;
            sh.Dr[lane * LS + j] = j < lane && rv ? (V)to_f32(d[k]) : (V)0;
            sh.Di[lane * LS + j] = 0;
            if (blk > 0) sh.Eb[lane * LS + j] = rv ? (V)to_f32(e[k]) : (V)0;
        }
    }
    diag_inverse_mx<V, BS, true>(sh.Dr, nullptr, sh.Eb, sh.Di, blk > 0, lane, wv);
    int jb = wv;
    if (jb < last) {
        load_tile_row<T, V, BS>(fv, LU, lda, rowc, (int64_t)jb * BS, n);
        cur.issue(tags, (int64_t)jb * BS + lane, true);
    }
    for (; jb < last; jb += 4) {
        const int nj = jb + 4;
        if (nj < last) {
            load_tile_row<T, V, BS>(fvn, LU, lda, rowc, (int64_t)nj * BS, n);
            nxt.issue(tags, (int64_t)nj * BS + lane, true);
        }
        cur.settle(tags, (int64_t)jb * BS + lane, true, epoch, &spins, flags, std::min(32, last - jb - 2));
        acc += row_times_lds<V, BS>(fv, cur.value(), sh.vb[wv], lane);
#pragma unroll
        for (int c = 0; c < BS; ++c) fv[c] = fvn[c];
        cur = nxt;
    }
    sh.part[wv][lane] = acc;
    __syncthreads();
    if (wv == 0) {
        V z = 0;
        if (rv) z = rhs(row) - ((sh.part[0][lane] + sh.part[1][lane]) + (sh.part[2][lane] + sh.part[3][lane]));
        V rr[BS];
        load_row<V, BS>(rr, sh.Di, lane);
        V w = row_times_lds<V, BS>(rr, z, sh.vb[0], lane);
        if (blk > 0) {
            // the only work left after the predecessor publishes: one product
            // with a row already in registers
            load_row<V, BS>(rr, sh.Dr, lane);
            lane_word<V> xp;
            xp.issue(tags, (int64_t)last * BS + lane, true);
            xp.template settle_ring<8>(tags, (int64_t)last * BS + lane, true, epoch, &spins, flags);
            w -= row_times_lds<V, BS>(rr, xp.value(), sh.vb[0], lane);
        }
        if (round_out) w = (V)to_f32((T)w);  // solution held in the factor precision
        if (rv) {
            tagged<V>::put(tags, row, w, epoch);
            out(row, w);
        }
    }
}

// Upper: blocks run from the last (nb - 1) to the first; tile blk + 1 enters
// through Mx = D^{-1} U_{b,b+1}.
template <typename T, typename V, int BS, typename Rhs, typename Out>
__device__ __forceinline__ void trsv_upper_block(TrsvLds<V, BS> &sh, int blk, int nb, int64_t n,
                                                 const T *__restrict__ LU, int64_t lda,
                                                 uint64_t *tags, uint32_t epoch,
                                                 int *__restrict__ flags, int round_out, Rhs rhs,
                                                 Out out)
{
    static_assert(BS == 64, "a wavefront spans one tile");
    constexpr int LS = TrsvLds<V, BS>::LS, PT = BS / 4;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t r0 = (int64_t)blk * BS;
    const int64_t row = r0 + lane;
    const bool rv = row < n;
    const int64_t rowc = rv ? row : 0;
    V acc = 0;
    int spins = 0;
    V fv[BS], fvn[BS];
    lane_word<V> cur, nxt;
    const int next = blk + 1;  // tiles jb > next go through the loop
    const bool has_next = next < nb;
    {
        T d[PT], e[PT];
#pragma unroll
        for (int k = 0; k < PT; ++k)
            d[k] = LU[rowc + std::min<int64_t>(r0 + wv + 4 * k, n - 1) * lda];
        if (has_next) {
#pragma unroll
            for (int k = 0; k < PT; ++k)
                e[k] = LU[rowc + std::min<int64_t>(r0 + BS + wv + 4 * k, n - 1) * lda];
        }
#pragma unroll
        for (int k = 0; k < PT; ++k) {
            const int j = wv + 4 * k;
            const bool in = rv && r0 + j < n;
            const V u = in ? (V)to_f32(d[k]) : (V)0;
            sh.Dr[lane * LS + j] = j > lane ? u : (V)0;
            if (j == lane) sh.rd[j] = in ? (V)1 / u : (V)1;
            sh.Di[lane * LS + j] = 0;
            if (has_next) sh.Eb[lane * LS + j] = rv && r0 + BS + j < n ? (V)to_f32(e[k]) : (V)0;
        }
    }
    diag_inverse_mx<V, BS, false>(sh.Dr, sh.rd, sh.Eb, sh.Di, has_next, lane, wv);
    int jb = nb - 1 - wv;
    if (jb > next) {
        load_tile_row<T, V, BS>(fv, LU, lda, rowc, (int64_t)jb * BS, n);
        cur.issue(tags, (int64_t)jb * BS + lane, (int64_t)jb * BS + lane < n);
    }
    for (; jb > next; jb -= 4) {
        const int nj = jb - 4;
        if (nj > next) {
            load_tile_row<T, V, BS>(fvn, LU, lda, rowc, (int64_t)nj * BS, n);
            nxt.issue(tags, (int64_t)nj * BS + lane, true);
        }
        const bool valid = (int64_t)jb * BS + lane < n;
        cur.settle(tags, (int64_t)jb * BS + lane, valid, epoch, &spins, flags, std::min(32, jb - next - 2));
        acc += row_times_lds<V, BS>(fv, valid ? cur.value() : (V)0, sh.vb[wv], lane);
#pragma unroll
        for (int c = 0; c < BS; ++c) fv[c] = fvn[c];
        cur = nxt;
    }
    sh.part[wv][lane] = acc;
    __syncthreads();
    if (wv == 0) {
        const V z = rv ? rhs(row) - ((sh.part[0][lane] + sh.part[1][lane]) + (sh.part[2][lane] + sh.part[3][lane])) : (V)0;
        V rr[BS];
        load_row<V, BS>(rr, sh.Di, lane);
        V w = row_times_lds<V, BS>(rr, z, sh.vb[0], lane);
        if (has_next) {
            load_row<V, BS>(rr, sh.Dr, lane);
            const bool valid = (int64_t)next * BS + lane < n;
            lane_word<V> xn;
            xn.issue(tags, (int64_t)next * BS + lane, valid);
            xn.template settle_ring<8>(tags, (int64_t)next * BS + lane, valid, epoch, &spins, flags);
            w -= row_times_lds<V, BS>(rr, valid ? xn.value() : (V)0, sh.vb[0], lane);
        }
        if (round_out) w = (V)to_f32((T)w);
        if (rv) {
            tagged<V>::put(tags, row, w, epoch);
            out(row, w);
        }
    }
}

// ------------------------------------------------------------ single solves
// y = L^{-1} (P b): L unit lower (below the diagonal of LU), perm[i] = the
// original row placed at position i (null = identity).
template <typename T, typename V, int BS>
__global__ __launch_bounds__(256) void k_trsv_lower(int64_t n, const T *__restrict__ LU, int64_t lda,
                                                    const int32_t *__restrict__ perm,
                                                    const V *__restrict__ b, V *__restrict__ y,
                                                    int *__restrict__ sync, uint32_t epoch,
                                                    int *__restrict__ flags, int round_out)
{
    __shared__ int s_blk;
    __shared__ TrsvLds<V, BS> sh;
    if (threadIdx.x == 0) s_blk = take_ticket(sync, epoch, gridDim.x);
    __syncthreads();
    trsv_lower_block<T, V, BS>(
        sh, s_blk, n, LU, lda, tag_words(sync), epoch, flags, round_out,
        [&](int64_t row) { return b[perm ? (int64_t)perm[row] : row]; },
        [&](int64_t row, V w) { y[row] = w; });
}

// x = S U^{-1} y with S = diag(colscale) (null = identity); other blocks read
// the unscaled solution (tagged).  With u non-null the solution is a
// refinement's correction and is added instead of stored: uprev = u, u += x
// (two launches a sweep less).
template <typename T, typename V, int BS>
__global__ __launch_bounds__(256) void k_trsv_upper(int64_t n, const T *__restrict__ LU, int64_t lda,
                                                    const V *__restrict__ yin,
                                                    const float *__restrict__ colscale,
                                                    V *__restrict__ x, V *__restrict__ u,
                                                    V *__restrict__ uprev, int *__restrict__ sync,
                                                    uint32_t epoch, int *__restrict__ flags,
                                                    int round_out)
{
    __shared__ int s_blk;
    __shared__ TrsvLds<V, BS> sh;
    const int nb = (int)((n + BS - 1) / BS);
    if (threadIdx.x == 0) s_blk = nb - 1 - take_ticket(sync, epoch, gridDim.x);
    __syncthreads();
    trsv_upper_block<T, V, BS>(
        sh, s_blk, nb, n, LU, lda, tag_words(sync), epoch, flags, round_out,
        [&](int64_t row) { return yin[row]; },
        [&](int64_t row, V w) {
#pragma clang fp contract(off)
            const V xi = colscale ? w * (V)colscale[row] : w;  // rounded before it is added
            if (!u) {
                x[row] = xi;
                return;
            }
            const V ui = u[row];
            uprev[row] = ui;
            u[row] = ui + xi;
        });
}

// ticket (4 ints, keeps the tag words 16-byte aligned) + 2 tag words per entry
size_t trsv_sync_ints(int64_t n) { return (size_t)(4 + 4 * n); }

template <typename T, typename V>
static hipError_t trsv_lower_t(int64_t n, const void *LU, int64_t lda, const int32_t *perm,
                               const V *b, V *y, int *sync, uint32_t epoch, int *flags,
                               hipStream_t s, int round_out = 0)
{
    const unsigned nb = (unsigned)((n + TRSV_BS - 1) / TRSV_BS);
    hipLaunchKernelGGL((k_trsv_lower<T, V, TRSV_BS>), dim3(nb), dim3(256), 0, s, n, (const T *)LU,
                       lda, perm, b, y, sync, epoch, flags, round_out);
    return hipGetLastError();
}

template <typename T, typename V>
static hipError_t trsv_upper_t(int64_t n, const void *LU, int64_t lda, const V *y,
                               const float *colscale, V *x, int *sync, uint32_t epoch, int *flags,
                               hipStream_t s, int round_out = 0, V *u = nullptr, V *uprev = nullptr)
{
    const unsigned nb = (unsigned)((n + TRSV_BS - 1) / TRSV_BS);
    hipLaunchKernelGGL((k_trsv_upper<T, V, TRSV_BS>), dim3(nb), dim3(256), 0, s, n, (const T *)LU,
                       lda, y, colscale, x, u, uprev, sync, epoch, flags, round_out);
    return hipGetLastError();
}

hipError_t launch_trsv_lower(int prec, int64_t n, const void *LU, int64_t lda, const int32_t *perm,
                             const float *b, float *y, int *sync, uint32_t epoch, int *flags,
                             hipStream_t s, int round_out)
{
    switch (prec) {
    case N3P_FP16: return trsv_lower_t<f16, float>(n, LU, lda, perm, b, y, sync, epoch, flags, s, round_out);
    case N3P_BF16: return trsv_lower_t<bf16, float>(n, LU, lda, perm, b, y, sync, epoch, flags, s, round_out);
    case N3P_FP32: return trsv_lower_t<float, float>(n, LU, lda, perm, b, y, sync, epoch, flags, s, round_out);
    case N3P_FP64: return trsv_lower_t<double, float>(n, LU, lda, perm, b, y, sync, epoch, flags, s, round_out);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_trsv_upper(int prec, int64_t n, const void *LU, int64_t lda, const float *y,
                             const float *colscale, float *x, int *sync, uint32_t epoch, int *flags,
                             hipStream_t s, int round_out, float *u, float *uprev)
{
    switch (prec) {
    case N3P_FP16: return trsv_upper_t<f16, float>(n, LU, lda, y, colscale, x, sync, epoch, flags, s, round_out, u, uprev);
    case N3P_BF16: return trsv_upper_t<bf16, float>(n, LU, lda, y, colscale, x, sync, epoch, flags, s, round_out, u, uprev);
    case N3P_FP32: return trsv_upper_t<float, float>(n, LU, lda, y, colscale, x, sync, epoch, flags, s, round_out, u, uprev);
    case N3P_FP64: return trsv_upper_t<double, float>(n, LU, lda, y, colscale, x, sync, epoch, flags, s, round_out, u, uprev);
    }
    return hipErrorInvalidValue;
}

// out = I_s^h(a * in): the scaled vector rounded to the factor type (held as
// FP32 values), the right-hand side of the low-precision solves of eq. (2.19)
template <typename T>
__global__ __launch_bounds__(256) void k_scale_round(int64_t n, const float *__restrict__ in, float a,
                                                     float *__restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) out[i] = to_f32((T)(in[i] * a));
}

hipError_t launch_scale_round(int prec, int64_t n, const float *in, float a, float *out, hipStream_t s)
{
    const unsigned g = (unsigned)((n + 255) / 256);
    switch (prec) {
    case N3P_FP16: hipLaunchKernelGGL(k_scale_round<f16>, dim3(g), dim3(256), 0, s, n, in, a, out); break;
    case N3P_BF16: hipLaunchKernelGGL(k_scale_round<bf16>, dim3(g), dim3(256), 0, s, n, in, a, out); break;
    case N3P_FP32:
    case N3P_FP64: hipLaunchKernelGGL(k_scale_round<float>, dim3(g), dim3(256), 0, s, n, in, a, out); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_trsv_lower_f64(int64_t n, const double *LU, int64_t lda, const int32_t *perm,
                                 const double *b, double *y, int *sync, uint32_t epoch, int *flags,
                                 hipStream_t s)
{
    return trsv_lower_t<double, double>(n, LU, lda, perm, b, y, sync, epoch, flags, s);
}

hipError_t launch_trsv_upper_f64(int64_t n, const double *LU, int64_t lda, const double *y,
                                 double *x, int *sync, uint32_t epoch, int *flags, hipStream_t s)
{
    return trsv_upper_t<double, double>(n, LU, lda, y, nullptr, x, sync, epoch, flags, s);
}

// ---------------------------------------------------------------- matvec
// r = b - A u (b may be null: r = sum), FP64 accumulation of FP32 data, two
// forms by size (launch_gemv_resid).
//
// One launch, n <= MV_ONE_N: a workgroup of 1024 threads owns MV_RB = 32 rows
// over all columns; a wavefront reads two columns' 128-byte pieces per load,
// each lane takes every 32nd column, eight loads in flight, and the 32
// column groups of a row are summed through LDS in a fixed order.  At these
// sizes the matrix comes from the caches and what bounds the product is how
// many loads are in flight: with one row (or four) per thread and 256
// columns in series the grid had ceil(n/1024) x ceil(n/256) workgroups of
// four wavefronts.  Measured, this form against that one (the reduction's
// launch included): n = 256 3.4 against 32 us, 1000 4.5 / 33, 2048 6.1 / 35,
// 4096 14.7 / 73 (4.6 TB/s).
// lane's part: rows [i0, i0 + MV_RB) of A (lda), us = u in LDS; the sum of
// row i0 + t is returned to threads t < MV_RB (0 to the others).
constexpr int MV_RB = 32, MV_NT = 1024, MV_UN = 8;
__device__ __forceinline__ double gemv_rows(int64_t n, const float *__restrict__ A, int64_t lda,
                                            const float *__restrict__ us, int64_t i0,
                                            double (*__restrict__ sh)[MV_RB])
{
    constexpr int G = MV_NT / MV_RB;
    const int t = threadIdx.x;
    const int64_t i = i0 + t % MV_RB;
    const float *ap = A + (i < n ? i : n - 1);  // rows past the end read row n - 1
    double s0 = 0.0, s1 = 0.0;
    int64_t j = t / MV_RB;
    for (; j + (int64_t)(MV_UN - 1) * G < n; j += (int64_t)MV_UN * G) {
        float a[MV_UN];
#pragma unroll
        for (int k = 0; k < MV_UN; ++k) a[k] = ap[(j + (int64_t)k * G) * lda];
#pragma unroll
        for (int k = 0; k < MV_UN; k += 2) {
            s0 += (double)a[k] * (double)us[j + k * G];
            s1 += (double)a[k + 1] * (double)us[j + (k + 1) * G];
        }
    }
    float a[MV_UN];
#pragma unroll
    for (int k = 0; k < MV_UN; ++k) {  // the last columns: index clamped, then left out
        const int64_t jj = j + (int64_t)k * G;
        a[k] = ap[(jj < n ? jj : n - 1) * lda];
    }
#pragma unroll
    for (int k = 0; k < MV_UN; ++k) {
        const int64_t jj = j + (int64_t)k * G;
        if (jj < n) s0 += (double)a[k] * (double)us[jj];
    }
    double s = s0 + s1;
    s += __shfl_xor(s, MV_RB);
    if ((t & 63) < MV_RB) sh[t >> 6][t & 63] = s;
    __syncthreads();
    double q = 0.0;
    if (t < MV_RB) {
#pragma unroll
        for (int w = 0; w < MV_NT / 64; ++w) q += sh[w][t];
    }
    return q;
}

constexpr int64_t MV_ONE_N = 4096;
__global__ __launch_bounds__(MV_NT) void k_gemv_rows(int64_t n, const float *__restrict__ A,
                                                     int64_t lda, const float *__restrict__ u,
                                                     const float *__restrict__ b,
                                                     float *__restrict__ r)
{
    __shared__ float us[MV_ONE_N];
    __shared__ double sh[MV_NT / 64][MV_RB];
    for (int64_t j = threadIdx.x; j < n; j += MV_NT) us[j] = u[j];
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * MV_RB + threadIdx.x;
    const double q = gemv_rows(n, A, lda, us, (int64_t)blockIdx.x * MV_RB, sh);
    if (threadIdx.x < MV_RB && i < n) r[i] = b ? (float)((double)b[i] - q) : (float)q;
}

// Larger n: partial sums over chunks of MV_CH columns, then their sum in a
// fixed order.  A workgroup of eight wavefronts owns 64 rows of one chunk,
// one row per lane, 32 columns per wavefront with 16 loads in flight (any
// alignment).  HBM-bound: n = 8192 44 us (6.2 TB/s, the sum included; 88 us
// with one or four rows per thread and the chunk's columns in series),
// 5003 26 / 32, 12000 101 / 169, 16384 188 / 206.
constexpr int MV_CH = 256, MV_CW = 8;
__global__ __launch_bounds__(MV_CW * 64) void k_gemv_part(int64_t n, const float *__restrict__ A,
                                                          int64_t lda, const float *__restrict__ u,
                                                          double *__restrict__ part)
{
    constexpr int PW = MV_CH / MV_CW, UN = 16;  // columns per wavefront, in flight
    __shared__ float ush[MV_CH];
    __shared__ double sh[MV_CW][64];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int64_t j0 = (int64_t)blockIdx.y * MV_CH;
    const int jn = (int)std::min<int64_t>(MV_CH, n - j0);
    if (t < MV_CH) ush[t] = t < jn ? u[j0 + t] : 0.0f;
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * 64 + lane;
    const float *ap = A + (i < n ? i : n - 1) + j0 * lda;
    double s0 = 0.0, s1 = 0.0;
#pragma unroll 1
    for (int c = w * PW; c < (w + 1) * PW; c += UN) {
        float a[UN];
#pragma unroll
        for (int k = 0; k < UN; ++k) a[k] = ap[(int64_t)std::min(c + k, jn - 1) * lda];
#pragma unroll
        for (int k = 0; k < UN; k += 2) {  // columns past the end: clamped and left out
            if (c + k < jn) s0 += (double)a[k] * (double)ush[c + k];
            if (c + k + 1 < jn) s1 += (double)a[k + 1] * (double)ush[c + k + 1];
        }
    }
    sh[w][lane] = s0 + s1;
    __syncthreads();
    if (t < 64 && i < n) {
        double q = 0.0;
#pragma unroll
        for (int k = 0; k < MV_CW; ++k) q += sh[k][t];
        part[(int64_t)blockIdx.y * n + i] = q;
    }
}

// the chunks of 32 rows per workgroup, eight chunks at a time (with one row
// per thread the chain over the chunks took 20 us at n = 16384; 6 us)
__global__ __launch_bounds__(256) void k_gemv_finish(int64_t n, int nch, const double *__restrict__ part,
                                                     const float *__restrict__ b, float *__restrict__ r)
{
    __shared__ double sh[8][32];
    const int t = threadIdx.x, g = t >> 5;
    const int64_t i = (int64_t)blockIdx.x * 32 + (t & 31);
    const int64_t ic = std::min<int64_t>(i, n - 1);
    double s = 0.0;
#pragma unroll 8
    for (int c = g; c < nch; c += 8) s += part[(int64_t)c * n + ic];
    sh[g][t & 31] = s;
    __syncthreads();
    if (t < 32 && i < n) {
        double q = 0.0;
#pragma unroll
        for (int k = 0; k < 8; ++k) q += sh[k][t];
        r[i] = b ? (float)((double)b[i] - q) : (float)q;
    }
}

hipError_t launch_gemv_resid(int64_t n, const float *A, int64_t lda, const float *u, const float *b,
                             float *r, double *part, hipStream_t s)
{
    // one launch up to MV_ONE_N: there both forms take the same time (14.7
    // and 14.0 us at 4096), and below it the second launch costs more than it
    // saves.  It writes rows of r while other workgroups still read u and A,
    // so a caller's r that overlaps either takes the two launches.
    const auto apart = [&](const float *p, int64_t len) { return r + n <= p || p + len <= r; };
    if (n <= MV_ONE_N && apart(u, n) && apart(A, (n - 1) * lda + n)) {
        hipLaunchKernelGGL(k_gemv_rows, dim3((unsigned)((n + MV_RB - 1) / MV_RB)), dim3(MV_NT), 0,
                           s, n, A, lda, u, b, r);
        return hipGetLastError();
    }
    const int nch = (int)((n + MV_CH - 1) / MV_CH);
    hipLaunchKernelGGL(k_gemv_part, dim3((unsigned)((n + 63) / 64), nch), dim3(MV_CW * 64), 0, s, n,
                       A, lda, u, part);
    hipLaunchKernelGGL(k_gemv_finish, dim3((unsigned)((n + 31) / 32)), dim3(256), 0, s, n, nch,
                       (const double *)part, b, r);
    return hipGetLastError();
}

hipError_t launch_gemv_f32(int64_t n, const float *A, int64_t lda, const float *v, float *y,
                           double *part, hipStream_t s)
{
    return launch_gemv_resid(n, A, lda, v, nullptr, y, part, s);
}

// ------------------------------------------------ allocation-free matvec
// Fixed scratch for the allocation-free form of r = b - A u: the FP64
// partial sums of one call, n * ceil(n / MV_CH) doubles for n <= GEMV_NOALLOC_MAX_N
// (8 MiB).  Each device holds its own copy at its own address until the
// process ends.  In host code `scratch` names a host-side stand-in, not device
// memory, so it is never passed to a kernel: the device address is looked up
// with hipGetSymbolAddress once per device (with that device current) and
// that pointer is what the kernels receive.
constexpr int64_t GEMV_NOALLOC_MAX_N = N3P_GEMV_NOALLOC_MAX_N;
constexpr size_t GEMV_NOALLOC_DOUBLES = (size_t)GEMV_NOALLOC_MAX_N * (GEMV_NOALLOC_MAX_N / MV_CH);
static_assert(GEMV_NOALLOC_MAX_N % MV_CH == 0, "scratch sized for whole column chunks");
static __device__ __align__(256) double scratch[GEMV_NOALLOC_DOUBLES];

constexpr int NOALLOC_MAX_DEVICES = 64;
static std::mutex g_scratch_mu;
static double *g_scratch_dev[NOALLOC_MAX_DEVICES];

static hipError_t noalloc_scratch(double **out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= NOALLOC_MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_dev[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!ptr) return hipErrorInvalidSymbol;
        g_scratch_dev[dev] = (double *)ptr;
    }
    *out = g_scratch_dev[dev];
    return hipSuccess;
}

hipError_t launch_gemv_resid_noalloc(int64_t n, const float *A, int64_t lda, const float *u,
                                     const float *b, float *r, hipStream_t s)
{
    if (n < 1 || n > GEMV_NOALLOC_MAX_N) return hipErrorInvalidValue;
    double *part = nullptr;
    const hipError_t e = noalloc_scratch(&part);
    if (e != hipSuccess) return e;
    return launch_gemv_resid(n, A, lda, u, b, r, part, s);
}

// ----------------------------------------------------------------- GMRES
// Modified Gram-Schmidt on one workgroup: for i = 0..j, h_i = <V_i, w>,
// w -= h_i V_i (sequentially, as MGS prescribes); h_{j+1} = ||w||,
// V_{j+1} = w / h_{j+1}.  Dots accumulate in FP64.
__device__ double block_sum_1024(double v, double *sh)
{
    const int t = threadIdx.x;
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if ((t & 63) == 0) sh[t >> 6] = v;
    __syncthreads();
    double s = 0.0;
    if (t == 0) {
        for (int w = 0; w < 16; ++w) s += sh[w];
        sh[16] = s;
    }
    __syncthreads();
    s = sh[16];
    __syncthreads();
    return s;
}

__global__ __launch_bounds__(1024) void k_mgs(int64_t n, float *__restrict__ V, int64_t ldv, int j,
                                              float *__restrict__ w, double *__restrict__ Hcol)
{
    __shared__ double sh[17];
    const int t = threadIdx.x;
    for (int i = 0; i <= j; ++i) {
        const float *vi = V + (int64_t)i * ldv;
        double d = 0.0;
        for (int64_t k = t; k < n; k += 1024) d += (double)vi[k] * (double)w[k];
        const double h = block_sum_1024(d, sh);
        const float hf = (float)h;
        for (int64_t k = t; k < n; k += 1024) w[k] -= hf * vi[k];
        if (t == 0) Hcol[i] = h;
        __syncthreads();
    }
    double q = 0.0;
    for (int64_t k = t; k < n; k += 1024) q += (double)w[k] * (double)w[k];
    const double hn = sqrt(block_sum_1024(q, sh));
    if (t == 0) Hcol[j + 1] = hn;
    float *vn = V + (int64_t)(j + 1) * ldv;
    const float inv = hn > 0.0 ? (float)(1.0 / hn) : 0.0f;
    for (int64_t k = t; k < n; k += 1024) vn[k] = w[k] * inv;
}

__global__ void k_krylov_update(int64_t n, const float *__restrict__ V, int64_t ldv, int k,
                                const double *__restrict__ y, float *__restrict__ d)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double s = 0.0;
    for (int q = 0; q < k; ++q) s += (double)V[(int64_t)q * ldv + i] * y[q];
    d[i] = (float)((double)d[i] + s);
}

hipError_t launch_mgs(int64_t n, float *V, int64_t ldv, int j, float *w, double *Hcol, hipStream_t s)
{
    hipLaunchKernelGGL(k_mgs, dim3(1), dim3(1024), 0, s, n, V, ldv, j, w, Hcol);
    return hipGetLastError();
}

hipError_t launch_krylov_update(int64_t n, const float *V, int64_t ldv, int k, const double *y,
                                float *d, hipStream_t s)
{
    hipLaunchKernelGGL(k_krylov_update, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, V,
                       ldv, k, y, d);
    return hipGetLastError();
}


// ====================================================== batched engine kernels
// The correction step of the IR algorithm of Section 2.2 for every refining
// slot: y = L^{-1} r, then z = U^{-1} y, d = S z (S the FP16 column scale),
// uprev = u, u += d, with the stored half-precision factors promoted to FP32
// as they are read (Section 2.3); LOWER, then upper, one launch each.
//
// Two forms by the request's size (never by what else is in the batch):
//
// At most B_SUBST_NP rows: one workgroup substitutes (b_substitute, in the
// lower launch).  A wavefront takes the diagonal block, a row a lane, while the
// other three hold the block's columns of the rows that it updates, so B_SUBST_NP
// is four wavefronts' rows.  With at most four blocks the chain is shorter than
// the inverses, tickets, hand-offs and second launch of the other form: 64
// requests of 200 rows 26 us a call against 48, of 64 rows 10 against 18.  At 512
// rows the other form is ahead (51 us for 32 requests, against 68 by one
// workgroup of sixteen wavefronts a request).
//
// More rows: the row blocks of the single solves.  A fixed grid takes them by
// ticket, all slots' first blocks, then all second ones, and so on: a block
// waits only on blocks of its own slot with smaller tickets, which running
// workgroups hold, so the waits end whatever the grid.  The published words
// and y lie in the slot's LT, which only the factorisation uses; k_b_ir_init
// clears the words each Newton step and the tags count the sweeps, so no tag
// repeats.  The tickets are cleared by the sweep's k_b_ir_check.
// These blocks multiply by explicit FP32 inverses of the diagonal blocks where
// the first form substitutes.  One solve with FP16 or BF16 factors of the
// H-equation's Jacobian at the solution, N = 512 to 4096 and c = 0.9 to 0.999999,
// is 0.8 to 1.3e-7 from 64 bits this way and 4e-7 to 1.6e-6 by row-by-row
// substitution: the shorter sums gain more than the inverses cost.
// With one workgroup per slot the 32 blocks of N = 2048 passed through one
// CU: 347 us a call for 32 requests of 128 to 2048 rows, now 98 for the two
// launches (240 for one workgroup with the substitution of a block beside the
// update by the one before it).
template <typename T>
__device__ __forceinline__ void b_substitute(const BDesc &q, float (&y)[B_SUBST_NP])
{
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int n = (int)q.n, Np = (int)q.Np;
    const T *__restrict__ A = (const T *)q.A;
    // one row of the 64 columns from b0, requested a block ahead
    T c[64], cn[64], dn;
    auto fetch = [&](int b0, int row) {
        const T *src = A + std::min(row, Np - 1) + (int64_t)b0 * Np;
#pragma unroll
        for (int k = 0; k < 64; ++k) cn[k] = src[(int64_t)k * Np];
        dn = A[(int64_t)(b0 + lane) * (Np + 1)];
    };
    auto update = [&](int b0, int row) {
        float acc = y[row];
#pragma unroll
        for (int k = 0; k < 64; ++k) acc -= to_f32(c[k]) * y[b0 + k];
        y[row] = acc;
    };
    y[t] = t < Np ? q.r[t] : 0.0f;
    fetch(0, t);
    __syncthreads();
#pragma unroll 1
    for (int b0 = 0; b0 < Np; b0 += 64) {  // forward, unit lower
#pragma unroll
        for (int k = 0; k < 64; ++k) c[k] = cn[k];
        // then the last block's upper half and the rows above it
        if (b0 + 64 < Np) fetch(b0 + 64, b0 + 64 + t);
        else fetch(b0, wv == 0 ? b0 + t : t - 64);
        if (wv == 0) {
            float yi = y[b0 + lane];
#pragma unroll
            for (int k = 0; k < 64; ++k) yi -= (lane > k ? to_f32(c[k]) : 0.0f) * lane_bcast(yi, k);
            y[b0 + lane] = yi;
        }
        __syncthreads();
        if (wv > 0 && b0 + t < Np) update(b0, b0 + t);
        __syncthreads();
    }
#pragma unroll 1
    for (int b0 = Np - 64; b0 >= 0; b0 -= 64) {  // backward, upper
        const T d = dn;
#pragma unroll
        for (int k = 0; k < 64; ++k) c[k] = cn[k];
        if (b0 > 0) fetch(b0 - 64, wv == 0 ? b0 - 64 + t : t - 64);
        if (wv == 0) {
            const float rd = 1.0f / to_f32(d);
            float yi = y[b0 + lane];
#pragma unroll
            for (int k = 63; k >= 0; --k) {
                if (lane == k) yi *= rd;
                yi -= (lane < k ? to_f32(c[k]) : 0.0f) * lane_bcast(yi, k);
            }
            y[b0 + lane] = yi;
        }
        __syncthreads();
        if (wv > 0 && t - 64 < b0) update(b0, t - 64);
        __syncthreads();
    }
    if (t < Np) {
        const float di = t < n ? (q.colscale ? y[t] * q.colscale[t] : y[t]) : 0.0f;
        const float ui = q.u[t];
        q.uprev[t] = ui;
        q.u[t] = ui + di;
    }
}

template <typename T, bool LOWER>
__global__ __launch_bounds__(256) void k_b_trsv(const BDesc *__restrict__ d,
                                                const BState *__restrict__ st, int nslots,
                                                int *__restrict__ ticket)
{
    constexpr int BS = 64, NLEV = B_MAX_NP / BS;
    static_assert(B_MAX_SLOTS <= 256 && NLEV <= 256, "one thread per slot and per level");
    __shared__ TrsvLds<float, BS> sh;
    __shared__ int nbs[B_MAX_SLOTS], order[B_MAX_SLOTS], lev[NLEV + 1], s_item;
    __shared__ float y_one[B_SUBST_NP];
    const int t = threadIdx.x;
    // blocks per slot (of the requests solved by blocks), the slots by falling number of blocks, and the number
    // of items on the levels before each
    int nb = 0;
    if (t < nslots) {
        const int on = st[t].ir_on != 0, nl = b_factor_leaves(d[t], st[t]);
        nb = on * nl * (NB_LEAF / BS);
        if (nb <= B_SUBST_NP / BS) nb = 0;
        nbs[t] = nb;
    }
    if constexpr (LOWER) {
        const int s = blockIdx.x;
        if (s < nslots && d[s].Np <= B_SUBST_NP && st[s].ir_on && b_factor_leaves(d[s], st[s]))
            b_substitute<T>(d[s], y_one);
    }
    if (!__syncthreads_or(nb)) return;
    int rank = 0, cnt = 0;
    for (int j = 0; j < nslots; ++j) {
        const int o = nbs[j];
        rank += o > nb || (o == nb && j < t);
        cnt += o > t;
    }
    if (t < nslots) order[rank] = t;
    if (t < NLEV) lev[t + 1] = cnt;
    __syncthreads();
    if (t == 0) {
        lev[0] = 0;
        for (int l = 0; l < NLEV; ++l) lev[l + 1] += lev[l];
    }
    __syncthreads();
    const int total = lev[NLEV];
    for (;;) {
        if (t == 0) s_item = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        const int item = s_item;
        if (item >= total) return;
        const int l = b_find(lev, NLEV, item);
        const int s = order[item - lev[l]];
        const BDesc &q = d[s];
        const int64_t Np = q.Np, n = q.n;
        uint64_t *tags = (uint64_t *)q.LT;
        float *y = (float *)(tags + Np);
        const uint32_t tag = 2 * (uint32_t)st[s].sweeps + (LOWER ? 1 : 2);
        if constexpr (LOWER) {
            trsv_lower_block<T, float, BS>(
                sh, l, Np, (const T *)q.A, Np, tags, tag, q.flags, 0,
                [&](int64_t row) { return q.r[row]; }, [&](int64_t row, float w) { y[row] = w; });
        } else {
            const int nblk = (int)(Np / BS);
            trsv_upper_block<T, float, BS>(
                sh, nblk - 1 - l, nblk, Np, (const T *)q.A, Np, tags, tag, q.flags, 0,
                [&](int64_t row) { return y[row]; },
                [&](int64_t row, float w) {
                    const float di = row < n ? (q.colscale ? w * q.colscale[row] : w) : 0.0f;
                    const float ui = q.u[row];
                    q.uprev[row] = ui;
                    q.u[row] = ui + di;
                });
        }
        __syncthreads();
    }
}

// r = b - J u with FP64 accumulation; items are MV_RB-row blocks of a slot
// (gemv_rows: a row's sum does not depend on the workgroup that takes it).
// With 256-row items, one row per thread, a request of 2048 rows had eight
// workgroups and 2048 columns in series: 112 us a call for 32 mixed requests.
__global__ __launch_bounds__(MV_NT) void k_b_gemv(const BDesc *__restrict__ d,
                                                  const BState *__restrict__ st, int nslots)
{
    __shared__ float us[B_MAX_NP];
    __shared__ int off[B_MAX_SLOTS + 1];
    __shared__ double sh[MV_NT / 64][MV_RB];
    const int total = b_offsets(nslots, off, [&](int s) {
        const int on = st[s].ir_on != 0, nl = b_factor_leaves(d[s], st[s]);
        return on * nl * (NB_LEAF / MV_RB);
    });
    const int t = threadIdx.x;
    for (int item = blockIdx.x; item < total; item += gridDim.x) {
        const int s = b_find(off, nslots, item);
        const BDesc &q = d[s];
        const int64_t n = q.n;
        for (int64_t j = t; j < n; j += MV_NT) us[j] = q.u[j];
        __syncthreads();
        const int64_t i0 = (int64_t)(item - off[s]) * MV_RB, i = i0 + t;
        const double sum = gemv_rows(n, q.J, n, us, i0, sh);
        if (t < MV_RB) q.r[i] = i < n ? (float)((double)q.b[i] - sum) : 0.0f;
        __syncthreads();
    }
}

// two workgroups fit a CU (256 registers a lane, 53 KB of LDS)
constexpr unsigned B_TRSV_GRID = 512;
static_assert(B_TRSV_GRID >= B_MAX_SLOTS, "a workgroup for every small request");
template <typename T>
static hipError_t b_solve_t(const BDesc *d, const BState *st, int nslots, bool blocks, int *tickets,
                            hipStream_t s)
{
    const dim3 grid(blocks ? B_TRSV_GRID : (unsigned)nslots);
    hipLaunchKernelGGL((k_b_trsv<T, true>), grid, dim3(256), 0, s, d, st, nslots, tickets);
    if (blocks)
        hipLaunchKernelGGL((k_b_trsv<T, false>), grid, dim3(256), 0, s, d, st, nslots, tickets + 1);
    return hipGetLastError();
}

hipError_t launch_b_solve(int prec, const BDesc *d, const BState *st, int nslots, bool blocks,
                          int *tickets, hipStream_t s)
{
    switch (prec) {
    case N3P_FP16: return b_solve_t<f16>(d, st, nslots, blocks, tickets, s);
    case N3P_BF16: return b_solve_t<bf16>(d, st, nslots, blocks, tickets, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_b_gemv(const BDesc *d, const BState *st, int nslots, int grid, hipStream_t s)
{
    hipLaunchKernelGGL(k_b_gemv, dim3(grid), dim3(MV_NT), 0, s, d, st, nslots);
    return hipGetLastError();
}

}  // namespace n3p
