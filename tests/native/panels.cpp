// Entry points for the tests of the pivoting path's single launches, linked
// with the library's own kernel objects: one leaf (the panel, then what is
// queued behind it) and an outer block's interchanges, on buffers and flags
// that the test prepares.
#include "n3p_internal.hpp"

using namespace n3p;

extern "C" {

// the exchange area, then the panel area
static size_t panel_offset(int prec, int64_t Np) { return (pivot_xch_bytes(prec, Np) + 255) / 256 * 256; }
N3P_API size_t panels_xch_bytes(int prec, int64_t Np)
{
    return panel_offset(prec, Np) + pivot_panel_bytes(prec, Np);
}
N3P_API int panels_nflags(void) { return NFLAGS; }
N3P_API int panels_flag_timeout(void) { return FLAG_TIMEOUT; }
N3P_API int panels_block_columns(void) { return NB_OUT; }

N3P_API int panels_leaf(int prec, int64_t Np, int64_t c0, int64_t k0, int64_t kend, void *A,
                        int64_t lda, int32_t *ipiv, void *LT, void *xch, int *flags, void *stream)
{
    hipStream_t s = (hipStream_t)stream;
    void *panel = (char *)xch + panel_offset(prec, Np);
    hipError_t e = launch_pivot_coop(prec, Np, c0, k0, A, lda, ipiv, LT, xch, panel, flags, s);
    if (e == hipSuccess) e = launch_gather_u12(prec, Np, c0, k0, kend, A, lda, LT, xch, panel, flags, s);
    return (int)e;
}

N3P_API int panels_block(int prec, int64_t Np, int64_t k0, int64_t kend, void *A, int64_t lda,
                         void *xch, void *stream)
{
    return (int)launch_gather_block(prec, Np, k0, kend, A, lda, xch, (hipStream_t)stream);
}

}  // extern "C"
