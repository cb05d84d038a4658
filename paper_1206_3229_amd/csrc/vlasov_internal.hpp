// Internal declarations shared by the host sources of the library (not part
// of the C ABI): the context, the workspace layout and small helpers.
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>

#include <memory>
#include <string>
#include <vector>

#include "vlasov.h"
#include "vlasov_kernels.hpp"

namespace vlasov_detail {

// Records the message of a failure for vlasov_last_error() and returns code.
int fail(int code, const std::string &msg);

#define HIP_TRY(expr)                                                                                   \
    do {                                                                                                \
        hipError_t e_ = (expr);                                                                         \
        if (e_ != hipSuccess)                                                                           \
            return ::vlasov_detail::fail(VLASOV_E_HIP, std::string(#expr) + ": " + hipGetErrorString(e_)); \
    } while (0)

constexpr size_t ALIGN = 256;
inline size_t align_up(size_t v) { return (v + ALIGN - 1) / ALIGN * ALIGN; }

// drift_threads of the default launch shape
constexpr int DRIFT_NT = 128;
// kick rows per thread (measured best on 4096^2: 16 for FP64, 32 for FP32)
template <typename T> constexpr int kick_rows() { return sizeof(T) == 8 ? 16 : 32; }
// fused kick and drift: default tile width and blocks
constexpr int KD_TW = 230, KD_RB = 2;
// 32-row tiles where the grid still gives at least this many of them, else
// 16-row tiles (twice the workgroups, to fill the chip)
constexpr int64_t KD_RB_MIN_TILES = 2048;
inline int default_kd_blocks(int64_t nx, int64_t nblk)
{
    return ((nx + KD_TW - 1) / KD_TW) * ((nblk + KD_RB - 1) / KD_RB) >= KD_RB_MIN_TILES ? KD_RB : 1;
}
// Sizes of f at which the drifts write their results through the L2s.
// From through_bytes() on: a kernel ends, and the next one starts, only once the lines its XCDs hold
// dirty are written back.  The fused kernel in steps of the sheet grid, written
// back -> through: FP64 128^2 6.5 -> 6.5 us, 512^2 6.8 -> 6.5, 1024^2 9.7 -> 9.1,
// 2048^2 18.4 -> 17.0, 4096^2 58.1 -> 55.8; FP32 (8 bytes a store) 256^2 5.8 ->
// 5.9, 512^2 5.9 -> 6.2, 724^2 6.3 -> 6.4, 1024^2 7.4 -> 7.4, 2048^2 13.6 -> 13.0,
// 4096^2 31.1 -> 30.8.  The density after it starts sooner as well (2048^2 ring
// 277 -> 264 us for 10 steps).
// Up to far_bytes(): the pair of buffers of larger grids does not fit in the 256
// MiB of the last-level cache, and the lines that two tiles share go to memory
// in two parts, one from each, unless the L2s put them together first.  Eight
// steps, written back / through, us: FP64 sheet 128 MiB of f 586 / 565, 136 MiB
// 625 / 632, 192 MiB 905 / 946; FP32 HMF 112 MiB 507 / 508, 128 MiB 708 / 726,
// 192 MiB 986 / 1071, 16384^2 4795 / 5516.
template <typename T> constexpr int64_t through_bytes() { return sizeof(T) == 8 ? int64_t(512) << 10 : int64_t(2) << 20; }
template <typename T> constexpr int64_t far_bytes() { return (sizeof(T) == 8 ? int64_t(132) : int64_t(120)) << 20; }
template <typename T> int64_t bytes_of_f(const vlasov_params &P) { return P.nx * P.np * (int64_t)sizeof(T); }
template <typename T> bool far_grid(const vlasov_params &P) { return bytes_of_f<T>(P) >= far_bytes<T>(); }
template <typename T> bool write_through(const vlasov_params &P)
{
    return bytes_of_f<T>(P) >= through_bytes<T>() && !far_grid<T>(P);
}
// Rows that the fused kernel's kick requests ahead.  FP64 four (4096^2 sheet,
// eight steps 568 us, 587 with two).  FP32 two, which is the faster by up to 5 % where f comes from
// the last-level cache (1024^2 sheet, eight steps 124 us, 130 with four), and
// four on far grids (16384^2 sheet 4771, 5447 with two).
template <typename T> constexpr int kd_pf(bool far = false) { return sizeof(T) == 8 || far ? 4 : 2; }
// rows per thread of the filter along p
constexpr int FILTER_R = 16;
// substeps of a step at most (the splittings of vlasov_splitting)
constexpr int MAX_SUB = 5;

// Sizes w_k of the substeps of one step (in units of dt); returns their number.
int split_weights(int scheme, double *w);

// Workspace layout (byte offsets, each 256-aligned).  The drift tables
// (drift_m, drift_w) hold one table per substep (np rows each), the fused
// kick-drift tables one per pair of consecutive substeps (kd_base nblk
// entries, kd_rel np entries each).
struct Layout {
    size_t drift_m, drift_w, kd_base, kd_rel, Fext, cs, sn, ringK, ringV, mxmy, hcount, gs_g;  // written at init
    size_t part, rho, F, hist, mom_out, mom_col, mom_phi;
    size_t total;
};

inline int64_t nblocks(int64_t np) { return (np + vk::ROWS_PER_BLOCK - 1) / vk::ROWS_PER_BLOCK; }

Layout layout_of(const vlasov_params &p);

// "" if the parameters are valid, else the reason.
std::string validate(const vlasov_params *p);

// "" if the spec of a generated initial condition is valid, else the reason.
std::string validate_ic(const vlasov_ic *ic);

}  // namespace vlasov_detail

struct vlasov_ctx {
    vlasov_params P;
    hipStream_t stream;
    size_t s;  // bytes per stored value
    char *f[2];
    int cur;
    char *ws;
    vlasov_detail::Layout L;
    double dx, dp;
    int64_t nblk;
    bool have_force;
    vlasov_tuning tune;  // launch shapes of the drift and kick
    // device whose static workspace this context holds (vlasov_init_static), or -1
    int static_dev = -1;
    // HIP graphs of gsteps whole steps (vlasov_set_graph; 0: none), captured on
    // cap_stream the first time they are needed, one per current buffer at the
    // start
    int gsteps = 0;
    hipStream_t cap_stream = nullptr;
    hipGraphExec_t gexec[2] = {nullptr, nullptr};
    int gcur_end[2] = {0, 0};  // current buffer after a replay
    // host copies kept for the tables of other tile heights
    std::vector<int64_t> h_mfull;  // drift foot offset per row, as the fused tables need it
    std::vector<int32_t> h_kd_base, h_kd_rel;
    // substeps of a step (splitting) and steps taken since init (filter schedule)
    int nsub;
    double wsub[vlasov_detail::MAX_SUB];
    int64_t steps_done;
    // largest spread of the drift offsets inside one tile of kd_rb blocks: of
    // the two half drifts after kick k (tables k, k+1 mod nsub; the fused
    // kernel runs up to 8 columns, on narrower tiles 56), and of the half
    // drift of table k alone (after the last kick of a call)
    int64_t kd_spread[vlasov_detail::MAX_SUB], kd_spread1[vlasov_detail::MAX_SUB];
    int kd_rb;
    // profiling
    bool prof;
    struct Rec {
        int kid;
        hipEvent_t a, b;
    };
    std::vector<Rec> recs;
    std::vector<hipEvent_t> pool;
    double ms[VLASOV_K_COUNT];
    int64_t cnt[VLASOV_K_COUNT];

    template <typename U> U *at(size_t off) const { return reinterpret_cast<U *>(ws + off); }
    // drift table of substep k
    const int32_t *dm(int k) const { return at<int32_t>(L.drift_m) + (size_t)k * (size_t)P.np; }
    const double4 *dw(int k) const { return at<double4>(L.drift_w) + (size_t)k * (size_t)P.np; }
    void *fcur() const { return f[cur]; }
    void *fnext() const { return f[cur ^ 1]; }
};

namespace vlasov_detail {
// Force array read by the kick: the caller's table for the EXTERNAL model.
inline const double *force_ptr(const vlasov_ctx *c)
{
    return c->at<double>(c->P.model == VLASOV_MODEL_EXTERNAL ? c->L.Fext : c->L.F);
}

inline hipEvent_t take_event(vlasov_ctx *c)
{
    if (!c->pool.empty()) {
        hipEvent_t e = c->pool.back();
        c->pool.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
}

// Launches a kernel on the context's stream.  When profiling is on, the
// launch carries its own start/stop events (recorded by the dispatch itself,
// so no extra packets sit between consecutive kernels).
template <typename... KArgs, typename... Args>
void launch_lds(vlasov_ctx *c, int kid, void (*kernel)(KArgs...), dim3 grid, dim3 block, size_t lds, Args... args)
{
    if (c->prof) {
        hipEvent_t a = take_event(c), b = take_event(c);
        if (a && b) {
            hipExtLaunchKernelGGL(kernel, grid, block, (uint32_t)lds, c->stream, a, b, 0, static_cast<KArgs>(args)...);
            c->recs.push_back({kid, a, b});
            return;
        }
    }
    kernel<<<grid, block, lds, c->stream>>>(static_cast<KArgs>(args)...);
}

template <typename... KArgs, typename... Args>
void launch(vlasov_ctx *c, int kid, void (*kernel)(KArgs...), dim3 grid, dim3 block, Args... args)
{
    launch_lds(c, kid, kernel, grid, block, 0, args...);
}

inline int check_launch(const char *what)
{
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(VLASOV_E_HIP, std::string(what) + ": " + hipGetErrorString(e));
    return VLASOV_OK;
}

// The current f as it is stored (synchronises), and its values as doubles.
int read_raw(vlasov_ctx *c, std::unique_ptr<char[]> &raw);
void widen(const char *raw, const vlasov_params &P, double *dst);
// Diagnostics in two parts: the kernels, and their result (synchronises).
int enqueue_moments(vlasov_ctx *c);
int fetch_moments(vlasov_ctx *c, vlasov_moments_t *out);

// Launchers (one translation unit per kernel family).  Each enqueues its
// kernel on the context's stream and, on success, makes the output buffer
// the current f.
// Half drift of table ta, then (tb >= 0) that of table tb, in one pass; with
// partials the density partial sums of the result.
template <typename T> int launch_drift(vlasov_ctx *c, int ta, int tb, bool partials);
// Kick of step size h with the last force.
template <typename T> int launch_kick(vlasov_ctx *c, double h);
// The filter along p; the kick of step size h followed by the filter.
template <typename T> int launch_filter(vlasov_ctx *c);
template <typename T> int launch_kick_filter(vlasov_ctx *c, double h);
// Global spline: half drift of table ta, then (tb >= 0) that of table tb, in one
// pass, and the partial sums of the result; kick.
template <typename T> int gs_drift_t(vlasov_ctx *c, int ta, int tb, bool partials);
template <typename T> int gs_kick_t(vlasov_ctx *c, double h);
// Kick of substep ta (step size h) fused with the half drifts of tables ta and
// ta + 1 mod nsub (pair), or with that of table ta alone; `spread` (at most
// KD_SPR_WIDE) is that of their offsets inside a tile.
template <typename T> int launch_kick_drift(vlasov_ctx *c, int ta, bool pair, int64_t spread, double h);
}  // namespace vlasov_detail

