// chol32.hip -- blocked right-looking FP32 Cholesky of Z on MFMA.
//
// Z is symmetric positive definite for distinct Euclidean points (Sections 2
// and 3.2), so Z = L L^T exists; this factor is computed in FP32 and used as
// the preconditioner of the FP64 refinement.  Panels of 512 columns (or 256, the
// tunable choice; 256 for a last, narrower one) are factored by one launch each
// (potrf.hip: 128 x 128 diagonal blocks, their inverses, the rows below, and L^T
// in the upper triangle).  They go in pairs: after the first panel a strip update
// brings the second one's columns up to date; after the second, one trailing
// update A22 -= L21 L21^T of both panels (K = 2 nb, lower tiles only) applies the
// pair to the rest.  A deep K amortises the load and store of each C tile over more
// matrix work.  Both run on the BF16 split image of the panels (gemm_split.hip), late
// strips on the FP32 instruction in 64-row tiles (twice the workgroups of 128-row
// ones, which keeps more CUs busy).  The inverses of the diagonal
// 128-blocks are kept (dinv) for the preconditioner's triangular solves.
#include "internal.hpp"

#include <algorithm>
#include <vector>

namespace mag {

// Rows above which the strip takes the split image, whose first half is then formed before
// it (5 us more in launches): up to 4096 rows the FP32 strip is one round of 64-row tiles,
// 23 us against 24-26 us on the image; above, 38 against 25 us at 4608 rows, 42 against 31 at 7680.
constexpr int64_t kSplitStrip = 4096;

// Factor the padded npad x npad FP32 matrix A (column-major, ld = npad) in place.
// timer (optional) records an event pair around every trailing update.
//
// Panels go in pairs (p, p+1): after panel p, only panel p+1's columns are
// updated by it (a strip, M x nb x nb); panel p+1 is factored; then one trailing
// update with K = 2 nb applies both panels to the rest.  Each tile of the large
// trailing block is read and written once per two panels.
void chol32_factor(hipStream_t s, float *A, int64_t npad, int64_t n, float *dinv, int *status,
                   FactorTimer *timer, int nb_max, void *img, void *work, long spin_limit)
{
    const int64_t kNb = (nb_max == 256) ? 256 : 512;
    int64_t k = 0;
    int panels = 0;
    launch_panel_begin(s, work, std::min<int64_t>(kNb, npad));
    while (k < npad) {
        const int64_t nb = std::min<int64_t>(kNb, npad - k);
        launch_panel(s, A, npad, k, nb, n, dinv, status, work, panels++, spin_limit);
        const int64_t k2 = k + nb;
        if (k2 >= npad) break;
        const int64_t nb2 = std::min<int64_t>(kNb, npad - k2);
        const int64_t below = npad - k2;
        const bool split = img && below > kSplitStrip;
        {
            // strip: panel p+1's columns (all rows from k2) by panel p; the tiles above
            // the 128-diagonal of its diagonal block are rewritten by its own panel launch
            float *C = A + k2 * npad + k2;
            const float *P = A + k * npad + k2;
            if (split) {
                launch_split(s, P, npad, below, nb, img, below, 0, 0);
                launch_strip_split(s, C, npad, img, below, nb2, nb);
            } else {
                launch_gemm_rows64(s, C, npad, P, npad, P, npad, below, nb2, nb);
            }
        }
        launch_panel(s, A, npad, k2, nb2, n, dinv, status, work, panels++, spin_limit);
        const int64_t k3 = k2 + nb2;
        const int64_t trail = npad - k3;
        if (trail > 0) {
            const int64_t K = nb + nb2;  // both panels, contiguous columns k .. k3-1
            float *C = A + k3 * npad + k3;
            const float *P = A + k * npad + k3;
            hipEvent_t e0 = nullptr, e1 = nullptr;
            if (timer) {
                if (timer->used + 2 > timer->ev.size()) {
                    for (int q = 0; q < 64; ++q) {
                        hipEvent_t e;
                        hipEventCreate(&e);
                        timer->ev.push_back(e);
                    }
                }
                e0 = timer->ev[timer->used++];
                e1 = timer->ev[timer->used++];
                // algorithmic flops of the trailing update restricted to the true n
                const int64_t nt = n - k3;
                timer->flops.push_back(nt > 0 ? (double)K * (double)nt * (double)(nt + 1) : 0.0);
                hipEventRecord(e0, s);
            }
            if (split) {
                launch_split(s, P + nb * npad, npad, trail, nb2, img, below, nb2, nb);
                launch_syrk_split(s, C, npad, img, below, nb2, trail, K);
            } else if (img) {
                launch_split(s, P, npad, trail, K, img, trail, 0, 0);
                launch_syrk_split(s, C, npad, img, trail, 0, trail, K);
            } else {
                launch_syrk_lower(s, C, npad, P, npad, trail, K);
            }
            if (timer) hipEventRecord(e1, s);
        }
        k = k3;
    }
}

size_t chol32_image_bytes(int64_t npad, int nb)
{
    const int64_t w = (nb == 256) ? 256 : 512;
    return npad > 2 * w ? split_image_bytes(npad - w, 2 * w) : 0;
}

int size_bucket(int64_t npad)
{
    int b = 0;
    while (b < 63 && ((int64_t)1 << b) < npad) ++b;
    return b;
}

int panel_width(const mag_ctx *ctx, int64_t npad)
{
    const int v = ctx ? ctx->tune_panel[size_bucket(npad)] : 0;
    return (v == 256 || v == 512) ? v : 512;
}

}  // namespace mag
