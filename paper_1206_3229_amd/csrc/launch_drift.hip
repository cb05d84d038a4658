// Kernel launchers of the library, one translation unit per kernel family
// (compiled in parallel); declared in vlasov_internal.hpp.
#include "vlasov_internal.hpp"

namespace vlasov_detail {

template <typename T, bool THROUGH, bool WIDE>
int launch_drift_by(vlasov_ctx *c, int ta, int tb, bool partials)
{
    const vlasov_params &P = c->P;
    const bool one = WIDE && tb < 0;
    const int tw = one ? vk::dr_width<1, WIDE>() : vk::dr_width<2, WIDE>(), nb = one ? 1 : default_kd_blocks(P.nx, c->nblk);
    const int ntx = (int)((P.nx + tw - 1) / tw), nty = (int)((c->nblk + nb - 1) / nb);
    const dim3 grid((unsigned)vk::xcd_grid(ntx, nty));
    const T *fin = (const T *)c->fcur();
    T *fout = (T *)c->fnext();
    const int32_t *dm1 = c->dm(ta), *dm2 = c->dm(tb >= 0 ? tb : ta);
    const double4 *dw1 = c->dw(ta), *dw2 = c->dw(tb >= 0 ? tb : ta);
    double *part = partials ? c->at<double>(c->L.part) : nullptr;
    const int nx = (int)P.nx, np = (int)P.np;
#define DRIFT_LAUNCH(KID, BX, NPASS)                                                                                   \
    launch(c, KID, vk::k_drift<T, BX, NPASS, THROUGH, WIDE>, grid, dim3(vk::dr_threads<T, NPASS, WIDE>()), fin, fout, \
           dm1, dm2, dw1, dw2, part, nx, np, nb, ntx, nty)
    if (P.bc_x == VLASOV_BC_PERIODIC) {
        if (tb >= 0) DRIFT_LAUNCH(VLASOV_K_DRIFT2, vk::BC_PERIODIC, 2); else DRIFT_LAUNCH(VLASOV_K_DRIFT, vk::BC_PERIODIC, 1);
    } else {
        if (tb >= 0) DRIFT_LAUNCH(VLASOV_K_DRIFT2, vk::BC_ZERO, 2); else DRIFT_LAUNCH(VLASOV_K_DRIFT, vk::BC_ZERO, 1);
    }
#undef DRIFT_LAUNCH
    int rc = check_launch("drift");
    if (rc == VLASOV_OK) c->cur ^= 1;
    return rc;
}

template <typename T>
int launch_drift(vlasov_ctx *c, int ta, int tb, bool partials)
{
    const bool wide = c->P.nx >= vk::KD_WIDE_MIN;
    if (write_through<T>(c->P))
        return wide ? launch_drift_by<T, true, true>(c, ta, tb, partials) : launch_drift_by<T, true, false>(c, ta, tb, partials);
    return wide ? launch_drift_by<T, false, true>(c, ta, tb, partials) : launch_drift_by<T, false, false>(c, ta, tb, partials);
}

template int launch_drift<float>(vlasov_ctx *, int, int, bool);
template int launch_drift<double>(vlasov_ctx *, int, int, bool);

}  // namespace vlasov_detail
