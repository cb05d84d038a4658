// Initial conditions of the paper's workloads (Sec. 4), generated on the
// device into a context's f (vlasov_generate_ic; the server's requests):
// waterbags, with the HMF map from (U, M0) to the half-widths, and the
// homogeneous Gaussian with a cos(x) seed.  Every one is normalised to unit
// mass on the grid with the raw values summed in index order, so that the
// result is a function of the specification alone.
#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "vlasov_internal.hpp"

using namespace vlasov_detail;

namespace {

// SplitMix64 (Steele, Lea and Flood 2014), counter-based: output k of the
// stream of `seed`.
constexpr uint64_t SM_GAMMA = 0x9E3779B97F4A7C15ull, SM_M1 = 0xBF58476D1CE4E5B9ull, SM_M2 = 0x94D049BB133111EBull;

__host__ __device__ inline uint64_t splitmix64(uint64_t seed, uint64_t k)
{
    uint64_t z = seed + (k + 1) * SM_GAMMA;
    z = (z ^ (z >> 30)) * SM_M1;
    z = (z ^ (z >> 27)) * SM_M2;
    return z ^ (z >> 31);
}

// Uniform double in [0, 1) from the top 53 bits.
__host__ __device__ inline double uniform01(uint64_t seed, uint64_t k)
{
    return (double)(splitmix64(seed, k) >> 11) * 0x1p-53;
}

struct Grid {
    int nx, np;
    double xmin, dx, pmin, dp;
};

struct Bag {
    double amp;
    uint64_t seed;
    // support: columns [i0, i0 + nc), rows [j0, j0 + nr)
    int i0, nc, j0, nr;
};

// The value of a support node.
__device__ __forceinline__ double bag_raw(const Grid &g, const Bag &w, int i, int j)
{
    if (w.amp == 0.0) return 1.0;
    const double eta = 2.0 * uniform01(w.seed, (uint64_t)j * (uint64_t)g.nx + (uint64_t)i) - 1.0;
    return 1.0 + w.amp * eta;
}

// Serial sums of the support rows from their first column (the zeros before
// and after it add nothing).  A workgroup sums 16 rows: four wavefronts form
// the values of the next 64 columns in LDS while lanes 0..15 of a fifth add
// those of the last 64, one row each in column order.  The additions of a row
// are one chain; 16 rows side by side and the values formed beside it leave
// that chain as the time.  Sheet waterbag on 2048^2: row sums and their sum 16 us
// (107 with every value of the grid stored first and one thread adding a
// row), the fill 11 us (25 with a division for the position of every value).
constexpr int IC_ROWS = 16, IC_COLS = 64, IC_NT = 320;

static __global__ __launch_bounds__(IC_NT) void k_ic_bag_rows(double *__restrict__ rows, Grid g, Bag w)
{
    __shared__ double buf[2][IC_COLS][IC_ROWS + 1];
    const int t = threadIdx.x, r = t & (IC_ROWS - 1);
    const int row = blockIdx.x * IC_ROWS + r;  // within the support
    const int j = w.j0 + min(row, w.nr - 1);
    const int ntile = (w.nc + IC_COLS - 1) / IC_COLS;
    double s = 0.0;
    for (int k = 0; k <= ntile; ++k) {
        if (t < 256) {
            if (k < ntile)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int c = (t >> 4) + 16 * q;
                    buf[k & 1][c][r] = bag_raw(g, w, w.i0 + IC_COLS * k + c, j);
                }
        } else if (k > 0 && t < 256 + IC_ROWS) {
            const int n = min(IC_COLS, w.nc - IC_COLS * (k - 1));
            for (int c0 = 0; c0 < n; c0 += 16) {
                double v[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) v[u] = buf[(k - 1) & 1][c0 + u][r];
#pragma unroll
                for (int u = 0; u < 16; ++u)
                    if (c0 + u < n) s = s + v[u];
            }
        }
        __syncthreads();
    }
    if (t >= 256 && t < 256 + IC_ROWS && row < w.nr) rows[row] = s;
}

// Serial sums of e_j c_i over i (one thread per row), the node factors c staged
// in LDS.
static __global__ __launch_bounds__(64) void k_ic_gauss_rows(const double *__restrict__ e, const double *__restrict__ c,
                                                             double *__restrict__ rows, Grid g)
{
    constexpr int CH = 1024;
    __shared__ double L[CH];
    const int j = blockIdx.x * 64 + threadIdx.x;
    const double ej = e[min(j, g.np - 1)];
    double s = 0.0;
    for (int i0 = 0; i0 < g.nx; i0 += CH) {
        const int n = min(CH, g.nx - i0);
        __syncthreads();
        for (int i = threadIdx.x; i < n; i += 64) L[i] = c[i0 + i];
        __syncthreads();
        int i = 0;
        for (; i + 16 <= n; i += 16) {
            double v[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) v[u] = ej * L[i + u];
#pragma unroll
            for (int u = 0; u < 16; ++u) s = s + v[u];
        }
        for (; i < n; ++i) s = s + ej * L[i];
    }
    if (j < g.np) rows[j] = s;
}

// The serial sum S of the n row sums and the divisor (S dx) dp: the sums pass
// through LDS, one thread adds them.
static __global__ __launch_bounds__(256) void k_ic_norm(const double *__restrict__ rows, double *__restrict__ norm,
                                                        Grid g, int n)
{
    constexpr int CH = 4096;
    __shared__ double L[CH];
    double s = 0.0;
    for (int k0 = 0; k0 < n; k0 += CH) {
        const int m = min(CH, n - k0);
        __syncthreads();
        for (int k = threadIdx.x; k < m; k += 256) L[k] = rows[k0 + k];
        __syncthreads();
        if (threadIdx.x == 0) {
            int k = 0;
            for (; k + 16 <= m; k += 16) {
                double v[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) v[u] = L[k + u];
#pragma unroll
                for (int u = 0; u < 16; ++u) s = s + v[u];
            }
            for (; k < m; ++k) s = s + L[k];
        }
    }
    if (threadIdx.x == 0) norm[0] = (s * g.dx) * g.dp;
}

// Four adjacent columns per thread, 256 columns by four rows per workgroup.
template <typename T>
__device__ __forceinline__ void ic_store(T *f, const Grid &g, int i, int j, const T (&v)[4])
{
    typedef T quad_t __attribute__((ext_vector_type(4), aligned(sizeof(T))));
    T *p = f + (size_t)j * (size_t)g.nx + i;
    if (i + 4 <= g.nx) {
        quad_t q;
        q.x = v[0];
        q.y = v[1];
        q.z = v[2];
        q.w = v[3];
        *reinterpret_cast<quad_t *>(p) = q;
    } else {
        for (int u = 0; u < 4; ++u)
            if (i + u < g.nx) p[u] = v[u];
    }
}

template <typename T>
static __global__ __launch_bounds__(256) void k_ic_bag_fill(T *__restrict__ f, const double *__restrict__ norm, Grid g,
                                                            Bag w)
{
    const int i = blockIdx.x * 256 + (threadIdx.x & 63) * 4;
    const double d = norm[0];
    for (int j = blockIdx.y * 4 + (threadIdx.x >> 6); j < g.np; j += gridDim.y * 4) {
        if (i >= g.nx) continue;
        T v[4] = {T(0), T(0), T(0), T(0)};
        if (j >= w.j0 && j < w.j0 + w.nr && i + 4 > w.i0 && i < w.i0 + w.nc)
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (i + u >= w.i0 && i + u < w.i0 + w.nc)
                    v[u] = (T)(bag_raw(g, w, i + u, j) / d);
        ic_store(f, g, i, j, v);
    }
}

template <typename T>
static __global__ __launch_bounds__(256) void k_ic_gauss_fill(T *__restrict__ f, const double *__restrict__ e,
                                                              const double *__restrict__ c,
                                                              const double *__restrict__ norm, Grid g)
{
    const int i = blockIdx.x * 256 + (threadIdx.x & 63) * 4;
    const double d = norm[0];
    for (int j = blockIdx.y * 4 + (threadIdx.x >> 6); j < g.np; j += gridDim.y * 4) {
        if (i >= g.nx) continue;
        const double ej = e[j];
        T v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = (T)((ej * c[min(i + u, g.nx - 1)]) / d);
        ic_store(f, g, i, j, v);
    }
}

// Nodes u_k = umin + k du with |u_k| <= half: first and count (they are
// adjacent, u_k grows with k), by the arithmetic of the nodes' definition.
void support(int n, double umin, double du, double half, int &first, int &count)
{
    first = 0;
    count = 0;
    for (int k = 0; k < n; ++k)
        if (fabs(umin + (double)k * du) <= half) {
            if (count == 0) first = k;
            ++count;
        }
}

// Half-widths of the HMF waterbag of magnetization M0 and energy U (Sec.
// 4.2): M0 = sin(theta0)/theta0, U = p0^2/6 + (1 - M0^2)/2.
bool hmf_halfwidths(double U, double M0, double &theta0, double &p0)
{
    if (!(M0 >= 0.0 && M0 < 1.0)) return false;
    const double kin = U - 0.5 * (1.0 - M0 * M0);
    if (!(kin >= 0.0)) return false;
    double lo = 0.0, hi = M_PI;
    for (int it = 0; it < 200; ++it) {
        const double mid = 0.5 * (lo + hi);
        const double val = mid > 0.0 ? sin(mid) / mid : 1.0;
        if (val > M0)
            lo = mid;
        else
            hi = mid;
        if (hi - lo <= 4e-16 * hi) break;
    }
    theta0 = 0.5 * (lo + hi);
    p0 = sqrt(6.0 * kin);
    return true;
}

}  // namespace

namespace vlasov_detail {

std::string validate_ic(const vlasov_ic *ic)
{
    if (!ic) return "NULL initial-condition spec";
    double t0, p0;
    switch (ic->kind) {
    case VLASOV_IC_WATERBAG:
        if (!std::isfinite(ic->a0) || !std::isfinite(ic->a1) || !std::isfinite(ic->amp))
            return "waterbag half-widths and noise must be finite";
        return "";
    case VLASOV_IC_WATERBAG_UM:
        if (!std::isfinite(ic->amp)) return "waterbag noise must be finite";
        if (!hmf_halfwidths(ic->a0, ic->a1, t0, p0)) return "waterbag (U, M0): need 0 <= M0 < 1 and U >= (1 - M0^2)/2";
        return "";
    case VLASOV_IC_GAUSSIAN:
        if (!(ic->a0 > 0.0) || !std::isfinite(ic->a0) || !(fabs(ic->amp) < 1.0)) return "gaussian: need T > 0 and |amp| < 1";
        return "";
    default:
        return "unknown initial-condition kind";
    }
}

}  // namespace vlasov_detail

extern "C" {

int vlasov_generate_ic(vlasov_ctx *c, const vlasov_ic *ic)
{
    if (!c || !ic) return fail(VLASOV_E_INVAL, "NULL argument");
    const vlasov_params &P = c->P;
    Grid g{(int)P.nx, (int)P.np, P.xmin, c->dx, P.pmin, c->dp};
    // scratch: row sums in the density partial sums (nblk nx >= np), the
    // divisor in rho; the Gaussian's node factors in the second f buffer (np
    // values) and the diagnostics columns (nx values)
    double *rows = c->at<double>(c->L.part);
    double *norm = c->at<double>(c->L.rho);
    const bool f32 = P.storage == VLASOV_F32;
    void *out = c->f[0];
    const dim3 fill((unsigned)((g.nx + 255) / 256), (unsigned)std::min((g.np + 3) / 4, 65535));
    const std::string why = validate_ic(ic);
    if (!why.empty()) return fail(VLASOV_E_INVAL, why);
    if (ic->kind == VLASOV_IC_WATERBAG || ic->kind == VLASOV_IC_WATERBAG_UM) {
        double x0 = ic->a0, p0 = ic->a1;
        if (ic->kind == VLASOV_IC_WATERBAG_UM) (void)hmf_halfwidths(ic->a0, ic->a1, x0, p0);
        Bag w{ic->amp, ic->seed, 0, 0, 0, 0};
        support(g.nx, g.xmin, g.dx, std::max(x0, 2.0 * c->dx), w.i0, w.nc);
        support(g.np, g.pmin, g.dp, std::max(p0, 2.0 * c->dp), w.j0, w.nr);
        if (w.nc == 0 || w.nr == 0) return fail(VLASOV_E_INVAL, "the initial condition has no mass on the grid");
        k_ic_bag_rows<<<(w.nr + IC_ROWS - 1) / IC_ROWS, IC_NT, 0, c->stream>>>(rows, g, w);
        k_ic_norm<<<1, 256, 0, c->stream>>>(rows, norm, g, w.nr);
        if (f32)
            k_ic_bag_fill<float><<<fill, 256, 0, c->stream>>>((float *)out, norm, g, w);
        else
            k_ic_bag_fill<double><<<fill, 256, 0, c->stream>>>((double *)out, norm, g, w);
    } else if (ic->kind == VLASOV_IC_GAUSSIAN) {
        const double T = ic->a0, A = ic->amp;
        const double phi = ic->seed == 0 ? 0.0 : 2.0 * M_PI * uniform01(ic->seed, 0);
        std::vector<double> e((size_t)P.np), cc((size_t)P.nx);
        for (int64_t j = 0; j < P.np; ++j) {
            const double v = P.pmin + (double)j * c->dp;
            e[(size_t)j] = exp(-(v * v) / (2.0 * T));
        }
        for (int64_t i = 0; i < P.nx; ++i) {
            const double x = P.xmin + (double)i * c->dx;
            cc[(size_t)i] = 1.0 + A * cos(x - phi);
        }
        double *de = reinterpret_cast<double *>(c->f[1]);
        double *dc = c->at<double>(c->L.mom_col);
        HIP_TRY(hipMemcpyAsync(de, e.data(), e.size() * sizeof(double), hipMemcpyHostToDevice, c->stream));
        HIP_TRY(hipMemcpyAsync(dc, cc.data(), cc.size() * sizeof(double), hipMemcpyHostToDevice, c->stream));
        k_ic_gauss_rows<<<(g.np + 63) / 64, 64, 0, c->stream>>>(de, dc, rows, g);
        k_ic_norm<<<1, 256, 0, c->stream>>>(rows, norm, g, g.np);
        if (f32)
            k_ic_gauss_fill<float><<<fill, 256, 0, c->stream>>>((float *)out, de, dc, norm, g);
        else
            k_ic_gauss_fill<double><<<fill, 256, 0, c->stream>>>((double *)out, de, dc, norm, g);
    }
    int rc = check_launch("initial condition");
    if (rc != VLASOV_OK) return rc;
    double d = 0.0;
    HIP_TRY(hipMemcpyAsync(&d, norm, sizeof d, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));  // also keeps the host tables alive until copied
    if (!(d > 0.0) || !std::isfinite(d)) return fail(VLASOV_E_INVAL, "the initial condition has no mass on the grid");
    c->cur = 0;
    return VLASOV_OK;
}

}  // extern "C"
