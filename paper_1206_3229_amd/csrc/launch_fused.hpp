// Launcher of the fused kick and drift kernel, shared by the translation units
// of the two storages.
#pragma once

#include "vlasov_internal.hpp"

namespace vlasov_detail {

template <typename T, int TW, int SPR, int NPASS, bool THROUGH, int PF>
int launch_kick_drift_w(vlasov_ctx *c, int kid, int ta, double h)
{
    using G = vk::KDGeom<TW, SPR>;
    constexpr int NT = NPASS == 2 ? G::NT : G::NT1;
    const vlasov_params &P = c->P;
    const int nb = c->kd_rb;
    const int ntx = (int)((P.nx + TW - 1) / TW), nty = (int)((c->nblk + nb - 1) / nb);
    const dim3 grid((unsigned)vk::xcd_grid(ntx, nty));
    const T *fin = (const T *)c->fcur();
    T *fout = (T *)c->fnext();
    const double *F = force_ptr(c);
    const int tb = (ta + 1) % c->nsub;
    const int32_t *dm1 = c->dm(ta), *dm2 = c->dm(tb);
    const double4 *dw1 = c->dw(ta), *dw2 = c->dw(tb);
    const int32_t *kbase = c->at<int32_t>(c->L.kd_base) + (size_t)ta * (size_t)c->nblk;
    const int32_t *krel = c->at<int32_t>(c->L.kd_rel) + (size_t)ta * (size_t)P.np;
    double *part = NPASS == 2 ? c->at<double>(c->L.part) : nullptr;
    const int nx = (int)P.nx, np = (int)P.np;
#define KD_LAUNCH(BX, BP)                                                                                      \
    launch(c, kid, vk::k_kick_drift<T, BX, BP, TW, SPR, PF, NPASS, THROUGH>, grid, dim3(NT), fin, fout, F, h, c->dp, \
           dm1, dm2, dw1, dw2, kbase, krel, part, nx, np, nb, ntx, nty)
    if (P.bc_x == VLASOV_BC_PERIODIC) {
        if (P.bc_p == VLASOV_BC_PERIODIC) KD_LAUNCH(vk::BC_PERIODIC, vk::BC_PERIODIC); else KD_LAUNCH(vk::BC_PERIODIC, vk::BC_ZERO);
    } else {
        if (P.bc_p == VLASOV_BC_PERIODIC) KD_LAUNCH(vk::BC_ZERO, vk::BC_PERIODIC); else KD_LAUNCH(vk::BC_ZERO, vk::BC_ZERO);
    }
#undef KD_LAUNCH
    int rc = check_launch("kick+drift");
    if (rc == VLASOV_OK) c->cur ^= 1;
    return rc;
}

template <typename T, bool THROUGH, int PF>
int launch_kick_drift_by(vlasov_ctx *c, int ta, bool pair, int64_t spread, double h)
{
    if (pair) {
        if (spread > vk::KD_SPR)
            return launch_kick_drift_w<T, vk::KD_TW_WIDE, vk::KD_SPR_WIDE, 2, THROUGH, PF>(c, VLASOV_K_KICK, ta, h);
        if (c->tune.kick_drift_width == 486)
            return launch_kick_drift_w<T, 486, vk::KD_SPR, 2, THROUGH, PF>(c, VLASOV_K_KICK_DRIFT2, ta, h);
        return launch_kick_drift_w<T, KD_TW, vk::KD_SPR, 2, THROUGH, PF>(c, VLASOV_K_KICK_DRIFT2, ta, h);
    }
    if (spread > vk::KD_SPR)
        return launch_kick_drift_w<T, vk::KD_TW_WIDE, vk::KD_SPR_WIDE, 1, THROUGH, PF>(c, VLASOV_K_KICK, ta, h);
    return launch_kick_drift_w<T, KD_TW, vk::KD_SPR, 1, THROUGH, PF>(c, VLASOV_K_KICK, ta, h);
}

template <typename T>
int launch_kick_drift(vlasov_ctx *c, int ta, bool pair, int64_t spread, double h)
{
    if (far_grid<T>(c->P)) return launch_kick_drift_by<T, false, kd_pf<T>(true)>(c, ta, pair, spread, h);
    return write_through<T>(c->P) ? launch_kick_drift_by<T, true, kd_pf<T>()>(c, ta, pair, spread, h)
                                  : launch_kick_drift_by<T, false, kd_pf<T>()>(c, ta, pair, spread, h);
}

}  // namespace vlasov_detail
