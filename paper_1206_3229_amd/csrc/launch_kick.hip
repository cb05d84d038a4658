// Kernel launchers of the library, one translation unit per kernel family
// (compiled in parallel); declared in vlasov_internal.hpp.
#include <algorithm>

#include "vlasov_internal.hpp"

namespace vlasov_detail {

template <typename T, int KR>
int launch_kick_r(vlasov_ctx *c, double h)
{
    const vlasov_params &P = c->P;
    const int ntx = (int)((P.nx + 255) / 256), nty = (int)((P.np + KR - 1) / KR);
    const dim3 grid((unsigned)vk::xcd_grid(ntx, nty));
    const T *fin = (const T *)c->fcur();
    T *fout = (T *)c->fnext();
    const double *F = force_ptr(c);
    if (P.bc_p == VLASOV_BC_PERIODIC)
        launch(c, VLASOV_K_KICK, vk::k_kick<T, vk::BC_PERIODIC, KR>, grid, dim3(256), fin, fout, F, h, c->dp,
               (int)P.nx, (int)P.np, ntx, nty);
    else
        launch(c, VLASOV_K_KICK, vk::k_kick<T, vk::BC_ZERO, KR>, grid, dim3(256), fin, fout, F, h, c->dp,
               (int)P.nx, (int)P.np, ntx, nty);
    int rc = check_launch("kick");
    if (rc == VLASOV_OK) c->cur ^= 1;
    return rc;
}

template <typename T>
int launch_kick(vlasov_ctx *c, double h)
{
    switch (c->tune.kick_rows) {
    case 8:
        return launch_kick_r<T, 8>(c, h);
    case 16:
        return launch_kick_r<T, 16>(c, h);
    default:
        return launch_kick_r<T, 32>(c, h);
    }
}

template <typename T>
int launch_filter(vlasov_ctx *c)
{
    const vlasov_params &P = c->P;
    const int ntx = (int)((P.nx + 255) / 256), nty = (int)((P.np + FILTER_R - 1) / FILTER_R);
    const dim3 grid((unsigned)vk::xcd_grid(ntx, nty));
    const T *fin = (const T *)c->fcur();
    T *fout = (T *)c->fnext();
    const double cf = P.filter_strength / 256.0;
    if (P.bc_p == VLASOV_BC_PERIODIC)
        launch(c, VLASOV_K_FILTER, vk::k_filter_p<T, vk::BC_PERIODIC, FILTER_R>, grid, dim3(256), fin, fout, cf,
               (int)P.nx, (int)P.np, ntx, nty);
    else
        launch(c, VLASOV_K_FILTER, vk::k_filter_p<T, vk::BC_ZERO, FILTER_R>, grid, dim3(256), fin, fout, cf,
               (int)P.nx, (int)P.np, ntx, nty);
    int rc = check_launch("filter");
    if (rc == VLASOV_OK) c->cur ^= 1;
    return rc;
}

template <typename T>
int launch_kick_filter(vlasov_ctx *c, double h)
{
    const vlasov_params &P = c->P;
    const int ntx = (int)((P.nx + 255) / 256), nty = (int)((P.np + FILTER_R - 1) / FILTER_R);
    const dim3 grid((unsigned)vk::xcd_grid(ntx, nty));
    const T *fin = (const T *)c->fcur();
    T *fout = (T *)c->fnext();
    const double cf = P.filter_strength / 256.0;
    if (P.bc_p == VLASOV_BC_PERIODIC)
        launch(c, VLASOV_K_FILTER, vk::k_kick_filter<T, vk::BC_PERIODIC, FILTER_R>, grid, dim3(256), fin, fout,
               force_ptr(c), h, c->dp, cf, (int)P.nx, (int)P.np, ntx, nty);
    else
        launch(c, VLASOV_K_FILTER, vk::k_kick_filter<T, vk::BC_ZERO, FILTER_R>, grid, dim3(256), fin, fout,
               force_ptr(c), h, c->dp, cf, (int)P.nx, (int)P.np, ntx, nty);
    int rc = check_launch("kick and filter");
    if (rc == VLASOV_OK) c->cur ^= 1;
    return rc;
}

// ---------------------------------------------------------------------------
// Global spline (eq. tridiagsys): half drifts of the rows in LDS, the kick down
// the columns.
// ---------------------------------------------------------------------------
// workgroups of the half drift that few rows are spread over: the CUs
constexpr int GS_MIN_WG = 256;
template <typename T, bool THROUGH>
int gs_drift_by(vlasov_ctx *c, int ta, int tb, bool partials)
{
    const vlasov_params &P = c->P;
    const T *fin = (const T *)c->fcur();
    T *fout = (T *)c->fnext();
    const int32_t *dm1 = c->dm(ta), *dm2 = c->dm(tb >= 0 ? tb : ta);
    const double4 *dw1 = c->dw(ta), *dw2 = c->dw(tb >= 0 ? tb : ta);
    const double *g = c->at<double>(c->L.gs_g);
    const int n = (int)P.nx, np = (int)P.np;
    // whole rows per workgroup: 128 threads of short rows (as far as 40 KB of
    // LDS hold them, and as the rows give every CU a workgroup), one long row.
    // Where rows are few, the threads without cells load and store (half drift
    // and partial sums, FP64, packed -> spread: 64^2 18 -> 10 us, 512^2 16 -> 13)
    const int tpl = vk::gs_threads(n, P.bc_x);
    const size_t row = (size_t)vk::gs_row(n, P.bc_x) * sizeof(T);
    const int lpw = std::max(1, std::min({128 / tpl, (int)(40960 / row), np / GS_MIN_WG})), grp = std::max(tpl, 128 / lpw);
    const dim3 grid((unsigned)((np + lpw - 1) / lpw)), block((unsigned)((grp * lpw + 63) / 64 * 64));
    const int kid = tb >= 0 ? VLASOV_K_DRIFT2 : VLASOV_K_DRIFT;
#define GS_ROWS(BC, NPASS)                                                                                          \
    launch_lds(c, kid, vk::k_gs_rows<T, BC, NPASS, THROUGH>, grid, block, row * (size_t)lpw, fin, fout, n, np, tpl, grp, lpw, dm1, \
               dw1, dm2, dw2, g)
    if (P.bc_x == VLASOV_BC_PERIODIC) {
        if (tb >= 0) GS_ROWS(vk::BC_PERIODIC, 2); else GS_ROWS(vk::BC_PERIODIC, 1);
    } else {
        if (tb >= 0) GS_ROWS(vk::BC_ZERO, 2); else GS_ROWS(vk::BC_ZERO, 1);
    }
#undef GS_ROWS
    int rc = check_launch("global-spline drift");
    if (rc) return rc;
    c->cur ^= 1;
    if (partials) {
        launch(c, kid, vk::k_partials<T>, dim3((unsigned)((P.nx + 255) / 256), (unsigned)c->nblk), dim3(256),
               (const T *)c->fcur(), c->at<double>(c->L.part), n, np);
        rc = check_launch("partial sums");
    }
    return rc;
}

template <typename T, bool THROUGH>
int gs_kick_by(vlasov_ctx *c, double h)
{
    const vlasov_params &P = c->P;
    const int nx = (int)P.nx, np = (int)P.np;
    const int ntx = (nx + 63) / 64, nty = (np + 4 * vk::GS_RK - 1) / (4 * vk::GS_RK);
    const dim3 grid((unsigned)vk::xcd_grid(ntx, nty));
    const T *fin = (const T *)c->fcur();
    T *fout = (T *)c->fnext();
    const double *g = c->at<double>(c->L.gs_g);
    if (P.bc_p == VLASOV_BC_PERIODIC)
        launch(c, VLASOV_K_KICK, vk::k_gs_cols<T, vk::BC_PERIODIC, THROUGH>, grid, dim3(256), fin, fout, nx, np, force_ptr(c), h,
               c->dp, g, ntx, nty);
    else
        launch(c, VLASOV_K_KICK, vk::k_gs_cols<T, vk::BC_ZERO, THROUGH>, grid, dim3(256), fin, fout, nx, np, force_ptr(c), h, c->dp,
               g, ntx, nty);
    int rc = check_launch("global-spline kick");
    if (rc == VLASOV_OK) c->cur ^= 1;
    return rc;
}

template <typename T>
int gs_drift_t(vlasov_ctx *c, int ta, int tb, bool partials)
{
    return write_through<T>(c->P) ? gs_drift_by<T, true>(c, ta, tb, partials) : gs_drift_by<T, false>(c, ta, tb, partials);
}

template <typename T>
int gs_kick_t(vlasov_ctx *c, double h)
{
    return write_through<T>(c->P) ? gs_kick_by<T, true>(c, h) : gs_kick_by<T, false>(c, h);
}

template int launch_kick<float>(vlasov_ctx *, double);
template int launch_kick<double>(vlasov_ctx *, double);
template int launch_filter<float>(vlasov_ctx *);
template int launch_filter<double>(vlasov_ctx *);
template int launch_kick_filter<float>(vlasov_ctx *, double);
template int launch_kick_filter<double>(vlasov_ctx *, double);
template int gs_drift_t<float>(vlasov_ctx *, int, int, bool);
template int gs_drift_t<double>(vlasov_ctx *, int, int, bool);
template int gs_kick_t<float>(vlasov_ctx *, double);
template int gs_kick_t<double>(vlasov_ctx *, double);

}  // namespace vlasov_detail
