// Device kernels of the split semi-Lagrangian Vlasov step for gfx950.
//
// Arithmetic contract (shared by every kernel here, compiled with
// -ffp-contract=off): products and sums round where written, fused
// multiply-adds appear only as explicit fma()/fmaf().  Every sum over an index
// of length n uses 64 interleaved running sums (term t in partial t mod 64,
// ascending t; the 64 lanes of a wavefront) combined by the xor butterfly
// d = 32, 16, ..., 1, so results do not depend on launch shapes.  Column sums
// over the momentum rows are serial inside blocks of 16 consecutive rows and
// then use that 64-way rule over the block index.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

namespace vk {

enum { BC_PERIODIC = 0, BC_ZERO = 1 };
constexpr int ROWS_PER_BLOCK = 16;  // rows of one density partial sum

// ---------------------------------------------------------------------------
// Eq. (findif): eighth-order centred second difference (without 1/du^2; the
// du^2 of the spline coefficients of eq. (splinecoeffs) cancels it).
// ---------------------------------------------------------------------------
template <typename T> struct FD;
template <> struct FD<double> {
    static constexpr double c0 = -205.0 / 72.0, c1 = 8.0 / 5.0, c2 = -1.0 / 5.0, c3 = 8.0 / 315.0,
                            c4 = -1.0 / 560.0;
};
template <> struct FD<float> {
    static constexpr float c0 = (float)(-205.0 / 72.0), c1 = (float)(8.0 / 5.0), c2 = (float)(-1.0 / 5.0),
                           c3 = (float)(8.0 / 315.0), c4 = (float)(-1.0 / 560.0);
};

__device__ __forceinline__ double vfma(double a, double b, double c) { return fma(a, b, c); }
__device__ __forceinline__ float vfma(float a, float b, float c) { return fmaf(a, b, c); }

// Marks loaded values as used here, after all of their loads, so that the
// compiler issues the loads together before any branch that follows (a load
// whose only use is conditional is otherwise moved into the branch, next to
// a wait for it).
template <typename T> __device__ __forceinline__ void keep_issued(T &v) { __asm__ __volatile__("" : "+v"(v)); }

// x points at the centre sample; reads x[-4..4].  Symmetric pairs first,
// accumulated from the outermost pair inwards.
template <typename T>
__device__ __forceinline__ T second_diff(const T *x)
{
    T s = FD<T>::c4 * (x[-4] + x[4]);
    s = vfma(FD<T>::c3, x[-3] + x[3], s);
    s = vfma(FD<T>::c2, x[-2] + x[2], s);
    s = vfma(FD<T>::c1, x[-1] + x[1], s);
    return vfma(FD<T>::c0, x[0], s);
}

// Eq. (splinegen) on the cell [k, k+1]: alpha f_k + beta f_k+1 + gamma D_k +
// delta D_k+1, accumulated in the order gamma, delta, beta, alpha.
template <typename T>
__device__ __forceinline__ T spline(T a, T b, T g, T d, T fk, T fk1, T Dk, T Dk1)
{
    T r = g * Dk;
    r = vfma(d, Dk1, r);
    r = vfma(b, fk1, r);
    return vfma(a, fk, r);
}

// ---------------------------------------------------------------------------
// Foot of the characteristic (Sec. 3): the new value at node i is the spline
// at i + xi cells, xi = -shift.  m = floor(xi), theta = xi - m (a rounded
// theta of 1 becomes 0 with m + 1); alpha = 1 - theta, beta = theta,
// gamma = (alpha^3 - alpha)/6, delta = (beta^3 - beta)/6.  A non-finite or
// huge shift gives m = 0 and NaN weights.
// ---------------------------------------------------------------------------
struct Foot {
    int64_t m;
    double a, b, g, d;
};

__host__ __device__ inline Foot foot_of_shift(double shift)
{
    Foot w;
    double xi = -shift;
    if (!(fabs(xi) < 2147483648.0)) {
        w.m = 0;
        w.a = w.b = w.g = w.d = __builtin_nan("");
        return w;
    }
    double fl = floor(xi);
    double th = xi - fl;
    w.m = (int64_t)fl;
    if (th >= 1.0) {
        th = 0.0;
        w.m += 1;
    }
    w.a = 1.0 - th;
    w.b = th;
    w.g = ((w.a * w.a) * w.a - w.a) / 6.0;
    w.d = ((w.b * w.b) * w.b - w.b) / 6.0;
    return w;
}

// Foot offset as used by the kernels: reduced to [0, n) on a periodic axis;
// clamped to +-(n + margin) with zero extension (beyond that every sample is 0;
// with the global spline, whose second derivatives reach 31 cells outside, at a
// larger margin).
constexpr int FOOT_MARGIN = 16, FOOT_MARGIN_GS = 64;
__host__ __device__ inline int32_t reduce_offset(int64_t m, int64_t n, int bc, int margin = FOOT_MARGIN)
{
    if (bc == BC_PERIODIC) {
        int64_t r = m % n;
        if (r < 0) r += n;
        return (int32_t)r;
    }
    int64_t lim = n + margin;
    return (int32_t)(m > lim ? lim : (m < -lim ? -lim : m));
}

__device__ __forceinline__ int wrap(int q, int n)
{
    int r = q % n;
    return r < 0 ? r + n : r;
}

// wrap() of a position that is mostly within one period of [0, n): the
// division only where it is not.
__device__ __forceinline__ int wrap_near(int q, int n)
{
    int r = q < 0 ? q + n : (q >= n ? q - n : q);
    if ((unsigned)r >= (unsigned)n) r = wrap(q, n);
    return r;
}

// reduce_offset() of a foot, whose m fits 32 bits (|xi| < 2^31).
template <int BC, int MARGIN = FOOT_MARGIN>
__device__ __forceinline__ int foot_offset(const Foot &ft, int n)
{
    const int m = (int)ft.m;
    return BC == BC_PERIODIC ? wrap_near(m, n) : min(max(m, -(n + MARGIN)), n + MARGIN);
}

// One sample of a line of n values (stride between samples `stride`) under
// the boundary rule of the axis.
template <typename T, int BC>
__device__ __forceinline__ T sample(const T *__restrict__ line, int q, int n, size_t stride)
{
    if (BC == BC_PERIODIC) return line[(size_t)wrap(q, n) * stride];
    return (q >= 0 && q < n) ? line[(size_t)q * stride] : T(0);
}

// Both halves of a pair of lanes swapped: in p the value of the lower lane of
// every pair 32 (or 16) lanes apart, in q that of the upper one.
template <int D>
__device__ __forceinline__ void spread_pairs(uint32_t v, uint32_t &p, uint32_t &q)
{
    const auto r = D == 32 ? __builtin_amdgcn_permlane32_swap(v, v, false, false)
                           : __builtin_amdgcn_permlane16_swap(v, v, false, false);
    p = r[0];
    q = r[1];
}
template <int D>
__device__ __forceinline__ double pair_sum(double v)
{
    uint32_t pl, ql, ph, qh;
    spread_pairs<D>((uint32_t)__double2loint(v), pl, ql);
    spread_pairs<D>((uint32_t)__double2hiint(v), ph, qh);
    return __hiloint2double((int)ph, (int)pl) + __hiloint2double((int)qh, (int)ql);
}
// v plus the value D lanes away in a row of 16 (which holds 16/(2 D) copies of
// the same 2 D values, so that a rotation by D is the exchange l ^ D).
template <int D>
__device__ __forceinline__ double row_sum(double v)
{
    constexpr int ROR = 0x120 + D;
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), ROR, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), ROR, 0xf, 0xf, true);
    return v + __hiloint2double(hi, lo);
}
// The xor butterfly d = 32, 16, ..., 1 over the 64 lanes.  The exchanges are
// register moves: through LDS each of the six waited for a round trip, and the
// density and force launches that end in this sum are short (a step at 128^2
// 12.0 -> 11.5 us, at 1024^2 16.4 -> 15.7).
__device__ __forceinline__ double wave_sum(double v)
{
    v = pair_sum<32>(v);
    v = pair_sum<16>(v);
    v = row_sum<8>(v);
    v = row_sum<4>(v);
    v = row_sum<2>(v);
    return row_sum<1>(v);
}

// Tile placement.  Workgroups are dispatched to the 8 XCDs of the chip in
// round-robin order of their linear id; each XCD is given a contiguous band of
// tile rows (x fastest inside the band) so that tiles sharing halo lines are
// served by the same L2.  Launch 8 * ceil(nty/8) * ntx workgroups.
constexpr int NXCD = 8;

__host__ __device__ inline int xcd_grid(int ntx, int nty) { return NXCD * ((nty + NXCD - 1) / NXCD) * ntx; }

__device__ __forceinline__ bool xcd_tile(int ntx, int nty, int &tx, int &ty)
{
    const int id = blockIdx.x;
    const int k = id / NXCD;
    const int per = (nty + NXCD - 1) / NXCD;
    ty = (id % NXCD) * per + k / ntx;
    tx = k % ntx;
    return ty < nty;
}

// ---------------------------------------------------------------------------
// Step 3 (eq. step3): kick along p, column i shifted by F_i dt/dp cells.  One
// thread per column and R consecutive output rows; the R + 9 samples of the
// column window are requested at once and held in registers (the lanes of a
// wavefront read adjacent columns of the same rows).
// ---------------------------------------------------------------------------
template <typename T, int BC, int R>
__device__ __forceinline__ void kick_tile(const T *__restrict__ fin, T *__restrict__ fout,
                                          const double *__restrict__ F, double dt, double dp, int nx, int np, int tx,
                                          int ty)
{
    const int i = tx * 256 + threadIdx.x;
    if (i >= nx) return;
    const int j0 = ty * R;
    const Foot ft = foot_of_shift((F[i] * dt) / dp);
    const int m = reduce_offset(ft.m, np, BC);
    const T a = (T)ft.a, b = (T)ft.b, g = (T)ft.g, d = (T)ft.d;
    const int base = j0 + m - 4;
    const T *col = fin + i;
    T w[R + 10];
#pragma unroll
    for (int s = 0; s < R + 10; ++s) w[s] = sample<T, BC>(col, base + s, np, (size_t)nx);
    T Dk = second_diff(w + 4);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const T Dk1 = second_diff(w + r + 5);
        const int j = j0 + r;
        if (j < np) fout[(size_t)j * nx + i] = spline(a, b, g, d, w[r + 4], w[r + 5], Dk, Dk1);
        Dk = Dk1;
    }
}

template <typename T, int BC, int R>
static __global__ __launch_bounds__(256) void k_kick(const T *__restrict__ fin, T *__restrict__ fout,
                                              const double *__restrict__ F, double dt, double dp, int nx, int np,
                                              int ntx, int nty)
{
    int tx, ty;
    if (!xcd_tile(ntx, nty, tx, ty)) return;
    kick_tile<T, BC, R>(fin, fout, F, dt, dp, nx, np, tx, ty);
}

// ---------------------------------------------------------------------------
// The filter along p, after the last kick of a filtered step (the filtering
// the conclusions name as an extension): out_j = f_j - c s_j with c =
// sigma/256 and s_j = sum_m b_m f_{j+m}, b the binomial weights (1, -8, 28,
// -56, 70, ...) of the eighth central difference, symmetric pairs added
// first and accumulated from the outermost pair inwards.  One thread per
// column and R consecutive rows, the R + 8 samples held in registers.
// ---------------------------------------------------------------------------
template <typename T, int BC, int R>
static __global__ __launch_bounds__(256) void k_filter_p(const T *__restrict__ fin, T *__restrict__ fout, double c,
                                                  int nx, int np, int ntx, int nty)
{
    int tx, ty;
    if (!xcd_tile(ntx, nty, tx, ty)) return;
    const int i = tx * 256 + threadIdx.x;
    if (i >= nx) return;
    const int j0 = ty * R;
    const T *col = fin + i;
    T w[R + 8];
#pragma unroll
    for (int s = 0; s < R + 8; ++s) w[s] = sample<T, BC>(col, j0 - 4 + s, np, (size_t)nx);
    const T cc = (T)c;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int j = j0 + r;
        const T *q = w + r + 4;
        T sm = q[-4] + q[4];
        sm = vfma(T(-8), q[-3] + q[3], sm);
        sm = vfma(T(28), q[-2] + q[2], sm);
        sm = vfma(T(-56), q[-1] + q[1], sm);
        sm = vfma(T(70), q[0], sm);
        if (j < np) fout[(size_t)j * nx + i] = vfma(-cc, sm, q[0]);
    }
}

// The kick of a filtered step followed by the filter, in one pass: each
// thread kicks rows j0 - 4 .. j0 + R + 3 of its column (the filter's window;
// rows outside the grid are zero with zero extension, wrapped otherwise)
// from R + 18 samples held in registers, then filters rows j0 .. j0 + R - 1.
// Every value is computed as by k_kick and k_filter_p, so the result is the
// same bit for bit.
// ---------------------------------------------------------------------------
template <typename T, int BC, int R>
static __global__ __launch_bounds__(256) void k_kick_filter(const T *__restrict__ fin, T *__restrict__ fout,
                                                     const double *__restrict__ F, double dt, double dp, double c,
                                                     int nx, int np, int ntx, int nty)
{
    int tx, ty;
    if (!xcd_tile(ntx, nty, tx, ty)) return;
    const int i = tx * 256 + threadIdx.x;
    if (i >= nx) return;
    const int j0 = ty * R;
    const Foot ft = foot_of_shift((F[i] * dt) / dp);
    const int m = reduce_offset(ft.m, np, BC);
    const T a = (T)ft.a, b = (T)ft.b, g = (T)ft.g, d = (T)ft.d;
    const int base = j0 - 8 + m;  // sample 0: row j0 - 4 + m - 4
    const T *col = fin + i;
    T w[R + 18];
#pragma unroll
    for (int s = 0; s < R + 18; ++s) w[s] = sample<T, BC>(col, base + s, np, (size_t)nx);
    // kicked rows j0 - 4 + u, u in [0, R + 8)
    T k[R + 8];
    T Dk = second_diff(w + 4);
#pragma unroll
    for (int u = 0; u < R + 8; ++u) {
        const T Dk1 = second_diff(w + u + 5);
        const T y = spline(a, b, g, d, w[u + 4], w[u + 5], Dk, Dk1);
        Dk = Dk1;
        const int row = j0 - 4 + u;
        k[u] = (BC == BC_PERIODIC || (row >= 0 && row < np)) ? y : T(0);
    }
    const T cc = (T)c;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const T *q = k + r + 4;
        T sm = q[-4] + q[4];
        sm = vfma(T(-8), q[-3] + q[3], sm);
        sm = vfma(T(28), q[-2] + q[2], sm);
        sm = vfma(T(-56), q[-1] + q[1], sm);
        sm = vfma(T(70), q[0], sm);
        const int j = j0 + r;
        if (j < np) fout[(size_t)j * nx + i] = vfma(-cc, sm, q[0]);
    }
}

// ---------------------------------------------------------------------------
// Step 3 fused with the half drifts that follow it: both (step 4 and step 1 of
// the next step) inside a call, step 4 alone after the last kick of a call.
// Once the force is known nothing global separates the kick of a row from its
// drifts, so one workgroup kicks the columns its drift windows need and drifts
// the kicked rows straight from LDS: f is read and written once for the two or
// three sweeps.  The arithmetic of every value is that of the separate kick
// and drifts, so results are identical bit for bit.
//
// Tile: nb consecutive density blocks (16 nb rows) by TW output columns.  The
// first-pass window of row j starts at column i0 + o_j - 8, o_j = m1_j + m2_j
// the sum of the row's two drift offsets; over the tile these windows lie in
// the KW = TW + 18 + SPR kicked columns starting at i0 + kbase (kbase = min_j
// o_j - 8, reduced mod nx on a periodic x axis), row j's window at offset
// krel_j = o_j - min o.  A grid whose tiles need krel > SPR takes the
// separate kernels.
//
// Work per interval of two rows (one barrier per interval, three intervals in
// flight), each part by waves of its own:
//   kick of rows r, r + 1: every lane kicks one column from a sliding register
//     window of its column (the kick of row r needs the samples r - 4 + m .. r
//     + 5 + m), loads requested PF rows ahead, and writes the kicked values to
//     the rows' LDS buffers;
//   first half drift of the two rows before them;
//   second half drift of the two rows before those, stored to HBM, and their
//     serial column sums over the block (density partial sums).
// A drift lane forms a run of four adjacent outputs (five stencils for four
// outputs), lanes 0..31 of a wave in the first row of the pair and lanes
// 32..63 in the second; the waves of a part share the runs of a row.
//
// All times here are of the launch in steps of the sheet grid (dt 0.01, calls of
// 20 steps), by its own events.
// What bounds it: small grids by the time of an interval in one wave (0.36 us;
// with every wave kicking and drifting in turn 0.5 us, hence waves of their own
// for each part); FP64 at 4096^2 by its loads and stores (56 us, without the
// drifts' arithmetic 52, without the kick's 52, with neither 49.5); FP32 there by
// VALU issue, 17.8 M wave-instructions of four cycles on 1024 SIMDs being all of
// its 70 000 cycles (30.5 us, 27.3, 28.5, and with no arithmetic 25.2).  Four
// rows an interval, loads 6 to 14 rows ahead, LDS reads an interval ahead and
// runs of two by twice the drifting waves were no faster.  Runs of four cost
// 15.25 operations an output and 7 LDS reads of 16 bytes for four (runs of two:
// 17.5, and 12); row weights stand in LDS and row offsets one per lane
// (v_readlane), where scalar loads between the barriers cost a wait each.  Every
// wave kicking and drifting -> parts, runs of four and stores through the L2s:
// 64^2 7.5 -> 6.3 us, 512^2 8.2 -> 6.5, 1024^2 10.4 -> 9.2, 2048^2 19.1 -> 16.8,
// 4096^2 60.1 -> 55.9; FP32 7.2 -> 5.5, 7.5 -> 5.9, 8.2 -> 7.2, 13.8 -> 13.0, 32.8
// -> 30.5.
// Registers: FP64 57 to 64, two spilled with periodic x and zero p; FP32 36 with
// periodic p, 54 to 58 with zero p; eight waves per SIMD in all.
// ---------------------------------------------------------------------------
constexpr int KD_SPR = 8;
// tiles for offsets that spread more (coarse p, fine x, long steps): the same
// kicked columns for fewer outputs
constexpr int KD_TW_WIDE = 182, KD_SPR_WIDE = 56;
// rows per barrier interval, and density blocks of a tile at most (the rows of
// a tile fit one per lane)
constexpr int KD_RPI = 2;
constexpr int KD_MAX_BLOCKS = 4;

// Where the drifted rows come from: kicked from f, or f itself (one value or 16
// bytes a lane).
enum { KD_KICK = 0, KD_LOAD = 1, KD_LOAD_WIDE = 2 };

// Geometry of a fused tile of TW columns whose rows' windows lie within SPR
// columns of slack: WK waves kick the KW = TW + 18 + SPR columns the windows
// need (one per lane), W1 waves run the first half drift (TW + 9 values per
// row) and W2 the second (TW outputs).  TW = 230 (4 + 2 + 2 waves) and 486 (8 +
// 4 + 4) with 8 columns of slack, and TW = 182 with 56, fill the kicking lanes.
template <int TW, int SPR = KD_SPR>
struct KDGeom {
    static constexpr int V = 4;                              // outputs per lane in the half drifts
    static constexpr int MIDN = TW + 9;                      // first-pass values per row
    static constexpr int NRUN1 = (MIDN + V - 1) / V;         // first-pass runs per row
    static constexpr int NRUN2 = (TW + V - 1) / V;           // second-pass runs per row
    static constexpr int KW = TW + 18 + SPR;                 // kicked columns per row
    static constexpr int WK = (KW + 63) / 64;
    static constexpr int W1 = (NRUN1 + 31) / 32, W2 = (NRUN2 + 31) / 32;
    static constexpr int NTK = 64 * WK, NT = 64 * (WK + W1 + W2);  // kicking lanes, threads
    static constexpr int NT1 = 64 * (WK + W2);                     // threads with one half drift
    static constexpr int R1 = (NRUN1 + W1 - 1) / W1, R2 = (NRUN2 + W2 - 1) / W2;  // runs per wave and row
    static constexpr int NBUF = 2 * KD_RPI;                  // rows in each LDS ring
    // Rows are held in groups of four values (KDRow).  Column c of the kicked
    // range is at slot c + pad, pad = -krel mod 4, so that every row's window
    // starts a group.
    static constexpr int NG = NTK / 4 + 4;                   // groups per row
    static constexpr int ROWLD = 4 * NG;                     // values per row
    // Part of wave w in workgroup `rot`: the kicking waves come first, so that
    // each SIMD gets kicking and drifting waves alike; the two drifts change
    // places from one workgroup to the next.  With one half drift the waves
    // past the kicking ones run it (those of a larger workgroup idle).  WL: the
    // waves that do the kicking ones' part.
    template <int NPASS, int WL> static __device__ __forceinline__ int part(int w, int rot)
    {
        if (w < WL) return w;
        w += WK - WL;
        if (NPASS == 1) return w + W1 < WK + W1 + W2 ? w + W1 : WK;
        const int d = w - WK + (rot & 1) * W1;
        return WK + (d < W1 + W2 ? d : d - (W1 + W2));
    }
    static_assert((SPR + 3) / 4 + NRUN1 + 3 <= NG && NRUN2 + 3 <= NG, "run reads stay in the row");
    static_assert(NG % 8 == 4, "the two halves of FP64 groups on distinct banks");
};

// A row of groups of four values in LDS.  FP32: contiguous, one 16-byte word
// per group.  FP64: the first pairs of all groups, then the second pairs, so
// that the lanes of a run read (lane u word u) touch consecutive 16-byte words.
template <typename T> struct KDRow;
template <> struct KDRow<float> {
    static __device__ __forceinline__ int at(int slot, int) { return slot; }
    template <int NG>
    static __device__ __forceinline__ void read(const float *row, int g, float (&x)[16])
    {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float4 v = reinterpret_cast<const float4 *>(row)[g + k];
            x[4 * k] = v.x;
            x[4 * k + 1] = v.y;
            x[4 * k + 2] = v.z;
            x[4 * k + 3] = v.w;
        }
    }
    template <int NG>
    static __device__ __forceinline__ void write(float *row, int g, const float (&o)[4])
    {
        reinterpret_cast<float4 *>(row)[g] = make_float4(o[0], o[1], o[2], o[3]);
    }
    static __device__ __forceinline__ void weights(const float *p, float (&w)[4])
    {
        const float4 v = *reinterpret_cast<const float4 *>(p);
        w[0] = v.x;
        w[1] = v.y;
        w[2] = v.z;
        w[3] = v.w;
    }
};
template <> struct KDRow<double> {
    static __device__ __forceinline__ int at(int slot, int ng) { return (slot >> 2) * 2 + (slot & 1) + (slot & 2) * ng; }
    template <int NG>
    static __device__ __forceinline__ void read(const double *row, int g, double (&x)[16])
    {
#pragma unroll
        for (int k = 0; k < 7; ++k) {  // samples 14 and 15 are not used
            const double2 v = reinterpret_cast<const double2 *>(row)[g + (k >> 1) + (k & 1) * NG];
            x[2 * k] = v.x;
            x[2 * k + 1] = v.y;
        }
        x[14] = x[15] = 0.0;
    }
    template <int NG>
    static __device__ __forceinline__ void write(double *row, int g, const double (&o)[4])
    {
        double2 *p = reinterpret_cast<double2 *>(row);
        p[g] = make_double2(o[0], o[1]);
        p[g + NG] = make_double2(o[2], o[3]);
    }
    static __device__ __forceinline__ void weights(const double *p, double (&w)[4])
    {
        const double2 v0 = reinterpret_cast<const double2 *>(p)[0], v1 = reinterpret_cast<const double2 *>(p)[1];
        w[0] = v0.x;
        w[1] = v0.y;
        w[2] = v1.x;
        w[3] = v1.y;
    }
};

// Four adjacent outputs from samples x[0 .. 13] (output k's cell starts at
// x[4 + k]).
template <typename T>
__device__ __forceinline__ void spline_run4(const T (&x)[16], T a, T b, T g, T d, T (&o)[4])
{
    T Dk = second_diff(x + 4);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const T Dk1 = second_diff(x + 5 + k);
        o[k] = spline(a, b, g, d, x[4 + k], x[5 + k], Dk, Dk1);
        Dk = Dk1;
    }
}

// Lanes 0..31 hold p, q of row a and lanes 32..63 those of row b.  Afterwards
// lanes 0..31 hold p of both rows (p: row a, q: row b) and lanes 32..63 q.
__device__ __forceinline__ void swap_halves(float &p, float &q)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(p), __float_as_uint(q), false, false);
    p = __uint_as_float(r[0]);
    q = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap_halves(double &p, double &q)
{
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(p), __double2loint(q), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(p), __double2hiint(q), false, false);
    p = __hiloint2double((int)hi[0], (int)lo[0]);
    q = __hiloint2double((int)hi[1], (int)lo[1]);
}

// Two adjacent values stored at any multiple of their own size (rows of an
// odd length).
template <typename T>
__device__ __forceinline__ void store2(T *p, T v0, T v1)
{
    typedef T pair_t __attribute__((ext_vector_type(2), aligned(sizeof(T))));
    pair_t v;
    v.x = v0;
    v.y = v1;
    *reinterpret_cast<pair_t *>(p) = v;
}

// store2() at `off` bytes into a row, written through the L2 of the XCD (no
// dirty lines for the end of the kernel to write back).
template <typename T>
__device__ __forceinline__ void store2_through(char *row, uint32_t off, T v0, T v1)
{
    constexpr int SC1 = 16;  // cache policy: device scope
    typedef T pair_t __attribute__((ext_vector_type(2)));
    typedef uint32_t words_t __attribute__((ext_vector_type(sizeof(T) / 2)));
    pair_t v;
    v.x = v0;
    v.y = v1;
    const auto r = __builtin_amdgcn_make_buffer_rsrc(row, 0, 0xffffffffu, 0x00027000);
    if constexpr (sizeof(T) == 8)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(words_t, v), r, off, 0, SC1);
    else
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(words_t, v), r, off, 0, SC1);
}

// One value, through the L2 or not.
template <bool THROUGH, typename T>
__device__ __forceinline__ void store1(T *p, T v)
{
    if constexpr (THROUGH)
        __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
        *p = v;
}

template <typename T>
struct KDTile {
    const T *fin;
    T *fout;
    const double *F;
    double dt, dp;
    const int32_t *dm1, *dm2;  // offsets of the half drifts in turn (the first one only with one pass)
    const double4 *dw1, *dw2;
    const int32_t *kbase, *krel;
    double *part;  // density partial sums of the result (NULL: none)
    int nx, np, nb, tx, ty;
    T *kbuf, *mbuf, *wtab;  // LDS: rings of NBUF rows of ROWLD values, 8 weights for each of the 16 nb rows
};

// Row of a tile that lane `lane` holds the offsets of (a tile has at most 64
// rows; lanes past the last one repeat it).
template <typename T>
__device__ __forceinline__ int kd_row(const KDTile<T> &a, int lane)
{
    const int j0 = a.ty * (ROWS_PER_BLOCK * a.nb);
    return min(j0 + lane, min(j0 + ROWS_PER_BLOCK * a.nb, a.np) - 1);
}

// Row offsets of a tile, one row per lane: the window's start in the kicked
// range (rel_v), and the first kicked column.
template <int NPASS, int BCX, typename T>
__device__ __forceinline__ void kd_rows(const KDTile<T> &a, int i0, int jl, int &rel_v, int &cL)
{
    if (NPASS == 2) {
        rel_v = a.krel[jl];
        cL = i0 + a.kbase[a.ty];
    } else {
        // offsets of the single half drift relative to their minimum over the
        // tile (the host checked that they spread by at most SPR columns; on a
        // periodic axis of nx >= 4 SPR they are known mod nx)
        const int dm = a.dm1[jl];
        const int ref = __builtin_amdgcn_readfirstlane(dm);
        int d = dm - ref;
        if (BCX == BC_PERIODIC) {
            d = 2 * d > a.nx ? d - a.nx : d;
            d = 2 * d < -a.nx ? d + a.nx : d;
        }
        int mn = d;
#pragma unroll
        for (int s = 32; s >= 1; s >>= 1) mn = min(mn, __shfl_xor(mn, s, 64));
        rel_v = d - mn;
        cL = i0 + ref + __builtin_amdgcn_readfirstlane(mn) - 4;
    }
}

// The kicking waves: lane t kicks column cL + t of every row of the tile.
template <typename T, int BCX, int BCP, int TW, int SPR, int PF, int NPASS>
__device__ __forceinline__ void kd_kick_part(const KDTile<T> &a, int t)
{
    using G = KDGeom<TW, SPR>;
    constexpr int R = ROWS_PER_BLOCK, LD = G::ROWLD, P = KD_RPI, NI = R / P, NB = G::NBUF;
    constexpr int NS = R + 10 + PF;  // window slots: samples of a block plus those requested ahead
    constexpr int LAG = NPASS;
    static_assert(PF % P == 0 && NS <= 32, "whole requests per interval, one mask bit per sample");
    const int nx = a.nx, np = a.np, i0 = a.tx * TW, j0 = a.ty * (R * a.nb);
    const int nblk = (min(R * a.nb, np - j0) + R - 1) / R;
    int rel_v, cL;
    kd_rows<NPASS, BCX>(a, i0, kd_row(a, t & 63), rel_v, cL);
    const int pad_v = 4 * ((rel_v + 3) >> 2) - rel_v;

    // Foot of the column's p shift (eq. step3), the spline weights, and the
    // row of the first sample.
    const int c = cL + t;
    int gc;
    bool colin = true, xin = true;
    if (BCX == BC_PERIODIC) {
        gc = wrap_near(c, nx);
    } else {
        gc = min(max(c, 0), nx - 1);
        colin = c >= 0 && c < nx;
        xin = cL >= 0 && cL + G::NTK <= nx;
    }
    const Foot ft = foot_of_shift((a.F[gc] * a.dt) / a.dp);
    const int m = foot_offset<BCP>(ft, np);
    const T ka = (T)ft.a, kb = (T)ft.b, kg = (T)ft.g, kd = (T)ft.d;
    // Samples are requested two rows at a time, from p0 and p1.  Where no
    // column of the wave needs a boundary rule in this tile (pin) both move by
    // two rows; otherwise the rows of the next request are wrapped (periodic)
    // or clamped, with bit s of `inside` saying that sample s lies in the grid.
    // The loads stand outside of that branch: in it, the compiler waited for
    // every outstanding load before the next request.
    int q0 = j0 + m - 4;
    if (BCP == BC_PERIODIC) q0 = wrap_near(q0, np);
    const size_t ld = (size_t)nx;
    const int pin = __builtin_amdgcn_readfirstlane((int)__all(q0 >= 0 && q0 + R * nblk + 10 + PF <= np));
    const T *fcol = a.fin + gc;
    uint32_t inside = 0;
    const T *p0, *p1;
    auto place = [&]() {
        if (BCP == BC_PERIODIC) {
            p0 = fcol + (size_t)q0 * ld;
            p1 = fcol + (size_t)(q0 + 1 < np ? q0 + 1 : 0) * ld;
        } else {
            p0 = fcol + (size_t)min(max(q0, 0), np - 1) * ld;
            p1 = fcol + (size_t)min(max(q0 + 1, 0), np - 1) * ld;
        }
    };
    place();
    T w[NS];
    auto request2 = [&](int s) {  // samples s, s + 1 of the window (of the current block)
        w[s] = *p0;
        w[s + 1] = *p1;
        if (pin) {
            p0 += 2 * ld;
            p1 += 2 * ld;
        } else {
            if (BCP != BC_PERIODIC) {
                inside |= (uint32_t)(q0 >= 0 && q0 < np) << s;
                inside |= (uint32_t)(q0 + 1 >= 0 && q0 + 1 < np) << (s + 1);
            }
            q0 += 2;
            if (BCP == BC_PERIODIC) q0 = q0 >= np ? q0 - np : q0;
            place();
        }
    };
    auto settle = [&](int s) {
        if (BCP != BC_PERIODIC)
            if (!pin) w[s] = (inside >> s & 1u) ? w[s] : T(0);
    };
#pragma unroll
    for (int s = 0; s < 10 + PF; s += 2) request2(s);
#pragma unroll
    for (int s = 0; s < 9; ++s) settle(s);
    T Dk = second_diff(w + 4);
    int pad = -1;
    T *dst = a.kbuf;  // LDS slot of the column in ring row 0, for the pad of the current row

    for (int blk = 0; blk < nblk; ++blk) {
        const bool more = blk + 1 < nblk;  // uniform
#pragma unroll
        for (int it = 0; it < NI; ++it) {
#pragma unroll
            for (int s = 0; s < P; ++s) {
                const int r = P * it + s;
                settle(r + 9);
                const T Dk1 = second_diff(w + r + 5);
                T y = spline(ka, kb, kg, kd, w[r + 4], w[r + 5], Dk, Dk1);
                Dk = Dk1;
                if (BCX == BC_ZERO && !xin) {
                    y = colin ? y : T(0);
                    __asm__ __volatile__("");  // a branch of the edge tiles, not a select in all
                }
                const int rp = __builtin_amdgcn_readlane(pad_v, R * blk + r);
                if (rp != pad) {  // uniform, changes a few times per tile at most
                    pad = rp;
                    dst = a.kbuf + KDRow<T>::at(t + pad, G::NG);
                }
                dst[(r & (NB - 1)) * LD] = y;
            }
            if (P * it + 10 + PF < R + 10 || more) request2(P * it + 10 + PF);
            __syncthreads();
        }
        // slide the window by one block: sample s + 16 becomes sample s
#pragma unroll
        for (int s = 0; s + R < NS; ++s) w[s] = w[s + R];
        inside >>= R;
    }
#pragma unroll
    for (int k = 0; k < LAG; ++k) __syncthreads();
}

// The loading waves of the drifts alone: lane t loads sample t of every row's
// own window, which starts at column i0 + o_j - 4 NPASS, PF rows ahead.
template <typename T, int BCX, int TW, int SPR, int NPASS>
__device__ __forceinline__ void kd_load_part(const KDTile<T> &a, int t)
{
    using G = KDGeom<TW, SPR>;
    constexpr int R = ROWS_PER_BLOCK, LD = G::ROWLD, P = KD_RPI, NI = R / P, NB = G::NBUF, PF = 8;
    static_assert(R % PF == 0 && PF % P == 0, "requested rows in the same registers block after block");
    const int nx = a.nx, np = a.np, i0 = a.tx * TW, j0 = a.ty * (R * a.nb);
    const int nblk = (min(R * a.nb, np - j0) + R - 1) / R;
    const int jl = kd_row(a, t & 63);
    int b_v = i0 + a.dm1[jl] + (NPASS == 2 ? a.dm2[jl] : 0) - 4 * NPASS;
    bool xin = true;
    int tm = t;  // periodic: sample t of a window that starts at b in [0, nx) is b + tm, less nx once past the end
    if (BCX == BC_PERIODIC) {
        b_v = wrap(b_v, nx);
        tm = t < nx ? t : wrap(t, nx);
    } else {
        xin = __all(b_v >= 0 && b_v + G::NTK <= nx);
    }
    const size_t ld = (size_t)nx;
    T v[PF];
    auto column = [&](int r) { return __builtin_amdgcn_readlane(b_v, r) + tm; };
    auto request = [&](int r, int slot) {
        int c = column(r);
        if (BCX == BC_PERIODIC)
            c = (int)min((unsigned)c, (unsigned)(c - nx));
        else
            c = min(max(c, 0), nx - 1);
        v[slot] = a.fin[(size_t)min(j0 + r, np - 1) * ld + (size_t)(unsigned)c];
    };
#pragma unroll
    for (int r = 0; r < PF; ++r) request(r, r);
    T *dst = a.kbuf + KDRow<T>::at(t, G::NG);
    for (int blk = 0; blk < nblk; ++blk) {
        const bool more = blk + 1 < nblk;  // uniform
#pragma unroll
        for (int it = 0; it < NI; ++it) {
#pragma unroll
            for (int s = 0; s < P; ++s) {
                const int r = P * it + s;
                T y = v[r % PF];
                if (BCX == BC_ZERO && !xin) {
                    const int c = column(R * blk + r);
                    y = c >= 0 && c < nx ? y : T(0);
                    __asm__ __volatile__("");  // a branch of the edge tiles, not a select in all
                }
                dst[(r & (NB - 1)) * LD] = y;
            }
            if (P * it + PF < R || more) {
#pragma unroll
                for (int s = 0; s < P; ++s) request(R * blk + P * it + s + PF, (P * it + s) % PF);
            }
            __syncthreads();
        }
    }
#pragma unroll
    for (int k = 0; k < NPASS; ++k) __syncthreads();
}

// The same with 16 bytes a lane and load, for lines of at least KD_WIDE_MIN
// columns: two rows at a time by KD_WIDE_WAVES waves, one a row in FP32, two in
// FP64.  EDGE (windows that pass an end of the grid): a lane's samples are taken
// from the nearest ones of the row and, on a periodic axis, from its first ones.
constexpr int KD_WIDE_MIN = 512;
template <typename T> constexpr int KD_WIDE_WAVES = 2 * 256 * (int)sizeof(T) / (64 * 16);
template <typename T, int BCX, int TW, int SPR, int NPASS, bool EDGE>
__device__ __forceinline__ void kd_load_rows(const KDTile<T> &a, int t, int b_v)
{
    using G = KDGeom<TW, SPR>;
    constexpr int R = ROWS_PER_BLOCK, LD = G::ROWLD, P = KD_RPI, NB = G::NBUF;
    constexpr int VEC = 16 / (int)sizeof(T), LPR = G::NTK / VEC, NI = R / P, PF = 4;
    static_assert(P * LPR == 64 * KD_WIDE_WAVES<T> && LPR % 64 == 0 && NI % PF == 0, "a row of the pair by whole waves");
    static_assert(KD_WIDE_MIN >= G::NTK + VEC, "a window passes the end of a line once");
    typedef T vec_t __attribute__((ext_vector_type(VEC)));
    typedef T load_t __attribute__((ext_vector_type(VEC), aligned(sizeof(T))));
    const int nx = a.nx, np = a.np, j0 = a.ty * (R * a.nb);
    const int nblk = (min(R * a.nb, np - j0) + R - 1) / R;
    const int q = __builtin_amdgcn_readfirstlane(t / LPR), l = t - q * LPR;  // row of the pair, place in it
    const size_t ld = (size_t)nx;
    vec_t v[PF], head[EDGE && BCX == BC_PERIODIC ? PF : 1];
    // first column of the lane's samples in row r, and the one they are loaded from
    auto column = [&](int r) { return __builtin_amdgcn_readlane(b_v, r) + VEC * l; };
    auto from = [&](int c) {
        if (!EDGE) return c;
        if (BCX == BC_PERIODIC) return c < nx ? min(c, nx - VEC) : c - nx;
        return min(max(c, 0), nx - VEC);
    };
    auto request = [&](int r, int slot) {
        const T *row = a.fin + (size_t)min(j0 + r, np - 1) * ld;
        v[slot] = *reinterpret_cast<const load_t *>(row + (unsigned)from(column(r)));
        if (EDGE && BCX == BC_PERIODIC) head[slot] = *reinterpret_cast<const load_t *>(row);
    };
    auto settle = [&](int r, int slot) {
        vec_t y = v[slot];
        if (EDGE) {
            const int c = column(r), d = BCX == BC_PERIODIC && c >= nx ? 0 : c - from(c);
            vec_t o;
#pragma unroll
            for (int k = 0; k < VEC; ++k) {
                T x = BCX == BC_PERIODIC ? y[k] : T(0);
#pragma unroll
                for (int e = BCX == BC_PERIODIC ? k + 1 : 0; e < (BCX == BC_PERIODIC ? k + VEC : VEC); ++e)
                    x = k + d == e ? (e < VEC ? y[e % VEC] : head[BCX == BC_PERIODIC ? slot : 0][e % VEC]) : x;
                o[k] = x;
            }
            y = o;
        }
        return y;
    };
#pragma unroll
    for (int it = 0; it < PF; ++it) request(P * it + q, it);
    // the lane's place in ring row 0: a group of four values in FP32, half a group in FP64
    vec_t *dst = reinterpret_cast<vec_t *>(a.kbuf) + (VEC == 4 ? l : (l >> 1) + (l & 1) * G::NG);
    // (the last block on its own: where its requests are left out by a branch in
    // the loop, the compiler waits for all outstanding ones at the loop's head)
    auto block = [&](int blk, auto last) {
#pragma unroll
        for (int it = 0; it < NI; ++it) {
            const int r = R * blk + P * it + q;
            dst[((P * it + q) & (NB - 1)) * (LD / VEC)] = settle(r, it % PF);
            if (!last.value || it + PF < NI) request(r + P * PF, it % PF);
            __syncthreads();
        }
    };
    for (int blk = 0; blk + 1 < nblk; ++blk) block(blk, std::false_type{});
    block(nblk - 1, std::true_type{});
#pragma unroll
    for (int k = 0; k < NPASS; ++k) __syncthreads();
}

template <typename T, int BCX, int TW, int SPR, int NPASS>
__device__ __forceinline__ void kd_load_wide(const KDTile<T> &a, int t)
{
    constexpr int NTK = KDGeom<TW, SPR>::NTK;
    const int jl = kd_row(a, t & 63);
    int b_v = a.tx * TW + a.dm1[jl] + (NPASS == 2 ? a.dm2[jl] : 0) - 4 * NPASS;
    if (BCX == BC_PERIODIC) b_v = wrap(b_v, a.nx);
    if (__all(b_v >= 0 && b_v + NTK <= a.nx))
        kd_load_rows<T, BCX, TW, SPR, NPASS, false>(a, t, b_v);
    else
        kd_load_rows<T, BCX, TW, SPR, NPASS, true>(a, t, b_v);
}

// The waves of the first half drift of a pair: wave w1 of W1.
template <typename T, int BCX, int TW, int SPR, int SRC>
__device__ __forceinline__ void kd_first_part(const KDTile<T> &a, int w1, int t)
{
    using G = KDGeom<TW, SPR>;
    constexpr int R = ROWS_PER_BLOCK, LD = G::ROWLD, P = KD_RPI, NB = G::NBUF;
    const int nx = a.nx, np = a.np, i0 = a.tx * TW, j0 = a.ty * (R * a.nb);
    const int nblk = (min(R * a.nb, np - j0) + R - 1) / R;
    const int lane = t & 63, l32 = lane & 31;
    const bool hi = lane >= 32;
    const int jl = kd_row(a, lane);
    const int st_v = SRC == KD_KICK ? (a.krel[jl] + 3) >> 2 : 0;  // group where the row's window starts
    int dm_v = 0;
    bool xin = true;  // no value of the tile lies outside the grid
    if (BCX == BC_ZERO) {
        dm_v = a.dm2[jl];
        const int lo = i0 + dm_v - 4;
        xin = __all(lo >= 0 && lo + 4 * G::NRUN1 <= nx);
    }
    const int u = min(G::R1 * w1 + min(l32, G::R1 - 1), G::NRUN1 - 1);  // lanes past the last run repeat it
    const T *src = a.kbuf + (hi ? LD : 0);
    T *dst = a.mbuf + (hi ? LD : 0);
    const T *wt = a.wtab + (hi ? 8 : 0);
    __syncthreads();
#pragma unroll 2
    for (int it = 0; it < nblk * (R / P); ++it) {
        const int qs = (P * it) & (NB - 1);  // ring slot of the pair's first row
        T x[16], wr[4], o[4];
        int g = u;
        if (SRC == KD_KICK) {
            const int sa = __builtin_amdgcn_readlane(st_v, P * it), sb = __builtin_amdgcn_readlane(st_v, P * it + 1);
            g += hi ? sb : sa;
        }
        KDRow<T>::template read<G::NG>(src + qs * LD, g, x);
        KDRow<T>::weights(wt, wr);
        wt += 8 * P;
        spline_run4<T>(x, wr[0], wr[1], wr[2], wr[3], o);
        if (BCX == BC_ZERO && !xin) {
            const int da = __builtin_amdgcn_readlane(dm_v, P * it), db = __builtin_amdgcn_readlane(dm_v, P * it + 1);
            const int q = i0 + (hi ? db : da) - 4 + 4 * u;
#pragma unroll
            for (int k = 0; k < 4; ++k) o[k] = q + k >= 0 && q + k < nx ? o[k] : T(0);
            __asm__ __volatile__("");  // a branch of the edge tiles, not a select in all
        }
        KDRow<T>::template write<G::NG>(dst + qs * LD, u, o);
        __syncthreads();
    }
    __syncthreads();
}

// The waves of the half drift whose result is stored: wave w2 of W2.  THROUGH:
// pairs are written through the L2 (single values and odd last rows are not).
template <typename T, int BCX, int TW, int SPR, int SRC, int NPASS, bool THROUGH>
__device__ __forceinline__ void kd_second_part(const KDTile<T> &a, int w2, int t)
{
    using G = KDGeom<TW, SPR>;
    constexpr int R = ROWS_PER_BLOCK, LD = G::ROWLD, P = KD_RPI, NB = G::NBUF, NI = R / P;
    constexpr int LAG = NPASS;
    constexpr bool ROWS = SRC == KD_KICK && NPASS == 1;  // windows start at their offset in the kicked range
    const int nx = a.nx, np = a.np, i0 = a.tx * TW, j0 = a.ty * (R * a.nb);
    const int nr = min(R * a.nb, np - j0), nblk = (nr + R - 1) / R;
    const int lane = t & 63, l32 = lane & 31;
    const bool hi = lane >= 32;
    int st_v = 0, cL;
    if (ROWS) {
        kd_rows<NPASS, BCX>(a, i0, kd_row(a, lane), st_v, cL);
        st_v = (st_v + 3) >> 2;
    }
    const int u = min(G::R2 * w2 + min(l32, G::R2 - 1), G::NRUN2 - 1);
    const int i = i0 + 4 * u + (hi ? 2 : 0);  // this lane stores columns i and i + 1
    const bool own = l32 < G::R2 && G::R2 * w2 + l32 < G::NRUN2;
    const int left = own ? min(i0 + TW, nx) - i : 0;
    const bool sums = a.part != nullptr;  // uniform
    const bool two = left >= 2, one = left == 1, anyone = __any(one);
    const T *src = (NPASS == 2 ? a.mbuf : a.kbuf) + (hi ? LD : 0);
    const T *wt = a.wtab + (hi ? 8 : 0) + (NPASS == 2 ? 4 : 0);
    const uint32_t io = (uint32_t)i * (uint32_t)sizeof(T), ios = (uint32_t)i * (uint32_t)sizeof(double);  // bytes
    const size_t ld = (size_t)nx, ldb = ld * sizeof(T);
    char *out = reinterpret_cast<char *>(a.fout + (size_t)j0 * ld);  // row stored next
#pragma unroll
    for (int k = 0; k < LAG; ++k) __syncthreads();
    for (int blk = 0; blk < nblk; ++blk) {
        double acc0 = 0.0, acc1 = 0.0;
#pragma unroll 2
        for (int it = 0; it < NI; ++it) {
            const int row = R * blk + P * it;
            const int qs = (P * it) & (NB - 1);
            T x[16], wr[4], o[4];
            int g = u;
            if (ROWS) {
                const int sa = __builtin_amdgcn_readlane(st_v, row), sb = __builtin_amdgcn_readlane(st_v, row + 1);
                g += hi ? sb : sa;
            }
            KDRow<T>::template read<G::NG>(src + qs * LD, g, x);
            KDRow<T>::weights(wt, wr);
            wt += 8 * P;
            spline_run4<T>(x, wr[0], wr[1], wr[2], wr[3], o);
            // o[0], o[1]: first row, o[2], o[3]: second row of the pair, of
            // columns i and i + 1
            swap_halves(o[0], o[2]);
            swap_halves(o[1], o[3]);
            T *outa = reinterpret_cast<T *>(out + io), *outb = reinterpret_cast<T *>(out + ldb + io);
            char *const row0 = out;
            out += 2 * ldb;
            if (row + 1 < nr) {
                if (two) {
                    if constexpr (THROUGH) {
                        store2_through<T>(row0, io, o[0], o[1]);
                        store2_through<T>(row0 + ldb, io, o[2], o[3]);
                    } else {
                        store2(outa, o[0], o[1]);
                        store2(outb, o[2], o[3]);
                    }
                }
                if (anyone)
                    if (one) {
                        outa[0] = o[0];
                        outb[0] = o[2];
                    }
                if (sums) {
                    acc0 = (acc0 + (double)o[0]) + (double)o[2];
                    acc1 = (acc1 + (double)o[1]) + (double)o[3];
                }
            } else if (row < nr) {
                if (two) store2(outa, o[0], o[1]);
                if (one) outa[0] = o[0];
                if (sums) {
                    acc0 = acc0 + (double)o[0];
                    acc1 = acc1 + (double)o[1];
                }
            }
            __syncthreads();
        }
        if (sums) {
            char *const sums0 = reinterpret_cast<char *>(a.part + (size_t)(a.ty * a.nb + blk) * ld);
            double *srow = reinterpret_cast<double *>(sums0 + ios);
            if (two) {
                if constexpr (THROUGH)
                    store2_through<double>(sums0, ios, acc0, acc1);
                else
                    store2(srow, acc0, acc1);
            }
            if (one) srow[0] = acc0;
        }
    }
}

// The waves without a part in a tile of one half drift.
template <int NPASS, typename T>
__device__ __forceinline__ void kd_no_part(const KDTile<T> &a)
{
    constexpr int R = ROWS_PER_BLOCK;
    const int nblk = (min(R * a.nb, a.np - a.ty * (R * a.nb)) + R - 1) / R;
    for (int k = 0; k < nblk * (R / KD_RPI) + NPASS; ++k) __syncthreads();
}

// One tile, by a workgroup of KDGeom::NT threads (or NT1 with one half drift;
// with KD_LOAD_WIDE fewer: dr_threads).
// SRC KD_KICK: the rows kicked, KD_LOAD: the rows of f (BCP, PF unused); then
// NPASS half drifts.  rot: number of the workgroup, t: of the thread in it.
template <typename T, int BCX, int BCP, int TW, int SPR, int PF, int SRC, int NPASS, bool THROUGH = false>
__device__ __forceinline__ void kick_drift_tile(const KDTile<T> &a, int rot, int t)
{
    using G = KDGeom<TW, SPR>;
    constexpr int R = ROWS_PER_BLOCK;
    constexpr int WL = SRC == KD_LOAD_WIDE ? KD_WIDE_WAVES<T> : G::WK;
    const int p = G::template part<NPASS, WL>(t >> 6, rot);
    if (p < G::WK) {
        if constexpr (SRC == KD_KICK)
            kd_kick_part<T, BCX, BCP, TW, SPR, PF, NPASS>(a, t);
        else if constexpr (SRC == KD_LOAD_WIDE)
            kd_load_wide<T, BCX, TW, SPR, NPASS>(a, t);
        else
            kd_load_part<T, BCX, TW, SPR, NPASS>(a, t);
    } else {
        // row weights, both passes of a row adjacent
        const int j0 = a.ty * (R * a.nb);
        const int n = 2 * R * ((min(R * a.nb, a.np - j0) + R - 1) / R);
        for (int k = t - 64 * WL; k < n; k += blockDim.x - 64 * WL) {
            const double4 w = (NPASS == 2 && (k & 1) ? a.dw2 : a.dw1)[min(j0 + (k >> 1), a.np - 1)];
            a.wtab[4 * k] = (T)w.x;
            a.wtab[4 * k + 1] = (T)w.y;
            a.wtab[4 * k + 2] = (T)w.z;
            a.wtab[4 * k + 3] = (T)w.w;
        }
        if (p >= G::WK + G::W1)
            kd_second_part<T, BCX, TW, SPR, SRC, NPASS, THROUGH>(a, p - G::WK - G::W1, t);
        else if (NPASS == 2)
            kd_first_part<T, BCX, TW, SPR, SRC>(a, p - G::WK, t);
        else
            kd_no_part<NPASS>(a);
    }
}

template <typename T, int BCX, int BCP, int TW, int SPR, int PF, int NPASS, bool THROUGH>
static __global__ __launch_bounds__((NPASS == 2 ? KDGeom<TW, SPR>::NT : KDGeom<TW, SPR>::NT1))
__attribute__((amdgpu_waves_per_eu(8)))
void k_kick_drift(
    const T *__restrict__ fin, T *__restrict__ fout, const double *__restrict__ F, double dt, double dp,
    const int32_t *__restrict__ dm1, const int32_t *__restrict__ dm2, const double4 *__restrict__ dw1,
    const double4 *__restrict__ dw2, const int32_t *__restrict__ kbase, const int32_t *__restrict__ krel,
    double *__restrict__ part, int nx, int np, int nb, int ntx, int nty)
{
    using G = KDGeom<TW, SPR>;
    __shared__ __attribute__((aligned(16))) T kbuf[G::NBUF * G::ROWLD];                    // ring of kicked rows
    __shared__ __attribute__((aligned(16))) T mbuf[NPASS == 2 ? G::NBUF * G::ROWLD : 4];  // of first-pass rows
    __shared__ __attribute__((aligned(16))) T wtab[8 * ROWS_PER_BLOCK * KD_MAX_BLOCKS];
    int tx, ty;
    if (!xcd_tile(ntx, nty, tx, ty)) return;
    const KDTile<T> a{fin, fout, F, dt, dp, dm1, dm2, dw1, dw2, kbase, krel, part, nx, np, nb, tx, ty, kbuf, mbuf, wtab};
    kick_drift_tile<T, BCX, BCP, TW, SPR, PF, KD_KICK, NPASS, THROUGH>(a, (int)blockIdx.x, (int)threadIdx.x);
}

// Steps 1 and 4 (eqs. step1, step4) without a kick before them: drift along x,
// row j shifted by the constant p_j tau/dx cells, once or (NPASS = 2, tables 1
// and 2) twice in turn; the tiles of the fused kernel with the rows' windows
// loaded instead of kicked.  Latency-bound on small grids (64^2 4.2 us; 11.5
// with a workgroup of two waves that waited for each row of an edge tile), near
// the copy rate on large ones.  It runs at the ends of a call, after every
// filtered kick, and for both half drifts of grids that cannot fuse.  WIDE
// (lines of KD_WIDE_MIN columns on): 16 bytes a load, and one half drift on
// tiles of 224 columns by one block, whose stores fill whole 128-byte lines
// where rows start on one.  One half drift, one value a load on tiles of 230 by
// two blocks -> wide, us: FP32 4096^2 25.7 -> 22.5, 2048^2 7.9 -> 7.5, 512 x
// 8192 10.2 -> 8.2; FP64 4096^2 48.0 -> 43.9, 2048^2 12.8 -> 11.7.  Two, on tiles of 230 by two blocks: FP32 4096^2 27.8 -> 26.2
// (tiles of 224 27.1, by one block 30), FP64 no change.
constexpr int DR_TW = 230;
template <int NPASS, bool WIDE> constexpr int dr_width() { return NPASS == 1 && WIDE ? 224 : DR_TW; }
template <typename T, int NPASS, bool WIDE>
constexpr int dr_threads()
{
    using G = KDGeom<dr_width<NPASS, WIDE>()>;
    return (NPASS == 2 ? G::NT : G::NT1) - (WIDE ? 64 * (G::WK - KD_WIDE_WAVES<T>) : 0);
}
template <typename T, int BCX, int NPASS, bool THROUGH, bool WIDE>
static __global__ __launch_bounds__((dr_threads<T, NPASS, WIDE>()))
__attribute__((amdgpu_waves_per_eu(8)))
void k_drift(
    const T *__restrict__ fin, T *__restrict__ fout, const int32_t *__restrict__ dm1, const int32_t *__restrict__ dm2,
    const double4 *__restrict__ dw1, const double4 *__restrict__ dw2, double *__restrict__ part, int nx, int np, int nb,
    int ntx, int nty)
{
    constexpr int TW = dr_width<NPASS, WIDE>();
    using G = KDGeom<TW>;
    __shared__ __attribute__((aligned(16))) T kbuf[G::NBUF * G::ROWLD];
    __shared__ __attribute__((aligned(16))) T mbuf[NPASS == 2 ? G::NBUF * G::ROWLD : 4];
    __shared__ __attribute__((aligned(16))) T wtab[8 * ROWS_PER_BLOCK * KD_MAX_BLOCKS];
    int tx, ty;
    if (!xcd_tile(ntx, nty, tx, ty)) return;
    const KDTile<T> a{fin, fout, nullptr, 0.0, 0.0, dm1, dm2, dw1, dw2, nullptr, nullptr, part, nx, np, nb, tx, ty, kbuf,
                      mbuf, wtab};
    kick_drift_tile<T, BCX, BC_PERIODIC, TW, KD_SPR, 2, WIDE ? KD_LOAD_WIDE : KD_LOAD, NPASS, THROUGH>(
        a, (int)blockIdx.x, (int)threadIdx.x);
}

// ---------------------------------------------------------------------------
// Eq. (tridiagsys): the global spline, the paper's baseline for the local f''.
// D_i = f''_i du^2 solves D_{i-1} + 4 D_i + D_{i+1} = 6 S_i with S_i =
// f_{i+1} - 2 f_i + f_{i-1} (on a periodic line, or on the line continued by
// zeros).  The (1, 4, 1) operator factors as -(1/r)(1 - r E)(1 - r E^-1),
// E the shift to the next node and r = sqrt(3) - 2 its root inside the unit
// circle, so D = -6 r x with y_i = S_i + r y_{i-1} (causal) and x_i = y_i +
// r x_{i+1} (anticausal): the convolution of S with sqrt(3) r^|k|.  Each
// thread runs both recursions over GS_R cells of a line in its registers,
// started GS_K nodes outside of them from 0 (|r|^GS_K is below FP64
// resolution), so a thread needs the samples from GS_K + 1 before its cells to
// GS_K + 1 after them and nothing from other threads.
// ---------------------------------------------------------------------------
constexpr int GS_K = 30, GS_R = 33, GS_MAX_N = 4096;

// Values of RC cells from the samples at(0 .. RC + 2 GS_K + 1), 31 before the
// first cell on (cell u lies between samples u + 31 and u + 32), left in y[0 ..
// RC).  `again` reads the samples of the cells a second time, so that they are
// not held in registers meanwhile.  fetch(s) comes before the samples s, s + 1,
// ..., s + RC, which are then asked for by their number and place in this group.
template <int RC, typename T, typename At, typename Again>
__device__ __forceinline__ void gs_cells(At at, Again again, T r, T cD, T a, T b, T g, T d, T (&y)[RC + GS_K])
{
    constexpr int S = RC + 2 * GS_K + 2, NB = RC + 1;
    T f0 = T(0), f1 = T(0), acc = T(0);
#pragma unroll
    for (int s0 = 0; s0 < S; s0 += NB) {
        at.fetch(s0);
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int s = s0 + u, e = s - 2;  // node of sample e + 1
            if (s < S) {
                const T f2 = at(s, u);
                if (e >= 0) acc = vfma(r, acc, (f0 + f2) - T(2) * f1);
                if (e >= GS_K) y[e - GS_K] = acc;
                f0 = f1;
                f1 = f2;
            }
        }
    }
    acc = T(0);
#pragma unroll
    for (int e = RC + GS_K - 1; e >= 0; --e) {
        acc = vfma(r, acc, y[e]);
        if (e <= RC) y[e] = cD * acc;
    }
    again.fetch(GS_K + 1);
    f0 = again(GS_K + 1, 0);
#pragma unroll
    for (int u = 0; u < RC; ++u) {
        f1 = again(GS_K + 2 + u, u + 1);
        y[u] = spline(a, b, g, d, f0, f1, y[u], y[u + 1]);
        f0 = f1;
    }
}

// Samples where they are needed, from p on, `ld` apart.
template <typename T>
struct GsDirect {
    const T *p;
    size_t ld;
    __device__ __forceinline__ void fetch(int) {}
    __device__ __forceinline__ T operator()(int s, int) const { return p[(size_t)s * ld]; }
};

// Samples of a column near the ends of the grid, from row q0 (in [0, np) on a
// periodic axis) on, NB at a time: with the boundary rule between two loads (a
// division, or a branch for the zero) each load waited for the one before it.
template <typename T, int BC, int NB>
struct GsEdge {
    const T *col;
    size_t ld;
    int q0, np;
    T buf[NB];
    __device__ __forceinline__ void fetch(int s)
    {
        int row = BC == BC_PERIODIC ? wrap_near(q0 + s, np) : 0;
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            if (BC != BC_PERIODIC) row = min(max(q0 + s + u, 0), np - 1);
            buf[u] = col[(size_t)(unsigned)row * ld];
            if (BC == BC_PERIODIC) row = row + 1 < np ? row + 1 : 0;
        }
#pragma unroll
        for (int u = 0; u < NB; ++u) keep_issued(buf[u]);
#pragma unroll
        for (int u = 0; u < NB; ++u)
            if (BC != BC_PERIODIC) buf[u] = (unsigned)(q0 + s + u) < (unsigned)np ? buf[u] : T(0);
    }
    __device__ __forceinline__ T operator()(int, int u) const { return buf[u]; }
};

// Threads per row of the drift (with zero extension 32 more cells on each
// side, where D decays to nothing) and samples of a row in LDS (GS_R of halo
// before the first cell and after the last one).  GS_R is odd, so that the
// threads of a row, GS_R cells apart, read distinct banks, and a zero-extended
// row of 2048 takes exactly one wavefront.
__host__ __device__ inline int gs_threads(int n, int bc) { return (n + (bc == BC_PERIODIC ? 0 : 64) + GS_R - 1) / GS_R; }
__host__ __device__ inline int gs_row(int n, int bc) { return GS_R * (gs_threads(n, bc) + 2); }

// The half drift of table 1 and (NPASS = 2) that of table 2, lpw rows per
// workgroup, the rows in LDS between the two.  A row is shifted by whole cells
// only when it is stored; in between, cells keep their place (place c of the
// second pass is column c - m1).  2048^2 FP64: 16 us, 21 for two half drifts
// (34 and 68 with both recursions through LDS, six barriers, and two workgroups
// per compute unit); the rows' traffic alone takes 11.  A row's `grp` threads
// load and store it, the first `tpl` of them have its cells: a short row has
// only two to four, which took up to 66 samples each from memory and back.
template <typename T, int BC, int NPASS, bool THROUGH>
static __global__ __launch_bounds__(256) void k_gs_rows(const T *__restrict__ fin, T *__restrict__ fout, int n, int lines,
                                                 int tpl, int grp, int lpw, const int32_t *__restrict__ dm1,
                                                 const double4 *__restrict__ dw1, const int32_t *__restrict__ dm2,
                                                 const double4 *__restrict__ dw2, const double *__restrict__ gcoef)
{
    extern __shared__ __attribute__((aligned(16))) char gs_lds[];
    constexpr int Z = BC == BC_PERIODIC ? 0 : 32;  // cells before column 0
    constexpr int H = GS_R;                        // sample e of the row is column e - H - Z
    const int l = threadIdx.x / grp, tt = threadIdx.x - l * grp;
    const int line = blockIdx.x * lpw + l;
    const bool mine = l < lpw && line < lines, cells = mine && tt < tpl;
    T *row = reinterpret_cast<T *>(gs_lds) + (size_t)min(l, lpw - 1) * gs_row(n, BC);
    const int NL = GS_R * (tpl + 2);
    if (mine) {
        const T *src = fin + (size_t)line * n;
        auto load = [&](auto batch) {  // samples of the row, `batch` a thread in flight
            constexpr int NB = decltype(batch)::value;
            for (int e0 = tt; e0 < NL; e0 += NB * grp) {
                T v[NB];
#pragma unroll
                for (int u = 0; u < NB; ++u) {
                    const int c = min(e0 + u * grp, NL - 1) - H - Z;
                    v[u] = BC == BC_PERIODIC ? src[wrap_near(c, n)] : src[min(max(c, 0), n - 1)];
                }
#pragma unroll
                for (int u = 0; u < NB; ++u) keep_issued(v[u]);
#pragma unroll
                for (int u = 0; u < NB; ++u) {
                    const int e = e0 + u * grp, c = e - H - Z;
                    if (e < NL) row[e] = BC == BC_PERIODIC || (c >= 0 && c < n) ? v[u] : T(0);
                }
            }
        };
        if (NL <= 4 * grp)
            load(std::integral_constant<int, 4>{});
        else
            load(std::integral_constant<int, 18>{});
    }
    __syncthreads();
    const T r = (T)gcoef[0], cD = (T)gcoef[1];
    T *mid = row + GS_R * min(tt, tpl - 1) + H;  // first cell of this thread
    int shift = 0;
#pragma unroll
    for (int pass = 0; pass < NPASS; ++pass) {
        T y[GS_R + GS_K];
        const int m = mine ? (pass == 0 ? dm1 : dm2)[line] : 0;
        if (cells) {
            const double4 w = (pass == 0 ? dw1 : dw2)[line];
            int o = 0;
            __asm__ __volatile__("" : "+v"(o));  // the second reads are reads
            const T *x = mid - GS_K - 1;
            gs_cells<GS_R>(GsDirect<T>{x, 1}, GsDirect<T>{x + o, 1}, r, cD, (T)w.x, (T)w.y, (T)w.z, (T)w.w, y);
        }
        shift += m;
        __syncthreads();
        if (cells) {
#pragma unroll
            for (int u = 0; u < GS_R; ++u) {
                T v = y[u];
                if (BC == BC_ZERO && pass + 1 < NPASS) {  // values outside the grid are zeros
                    const int i = GS_R * tt + u - Z - m;
                    v = i >= 0 && i < n ? v : T(0);
                }
                mid[u] = v;
            }
        }
        __syncthreads();
        if (BC == BC_PERIODIC && pass + 1 < NPASS) {  // the halos again
            if (mine)
                for (int e = tt; e < NL - n; e += grp) {
                    const int h = e < H ? e : e + n;
                    row[h] = row[wrap(h - H, n) + H];
                }
            __syncthreads();
        }
    }
    if (mine) {
        T *dst = fout + (size_t)line * n;
        if (BC == BC_PERIODIC) shift = wrap(shift, n);
        for (int i = tt; i < n; i += grp) {
            int c = i + shift;
            if (BC == BC_PERIODIC) {
                c = c >= n ? c - n : c;
                store1<THROUGH>(dst + i, row[c + H]);
            } else {
                store1<THROUGH>(dst + i, c >= -Z && c < GS_R * tpl - Z ? row[c + Z + H] : T(0));
            }
        }
    }
}

// The kick: one thread per column and GS_RK rows, the samples read down the
// column (the lanes of a wavefront read adjacent columns of the same rows, and
// the rows that two chunks share come from the caches).  Small grids take the
// time of one wave, near the ends of the grid three groups of loads and their
// arithmetic; large ones the reads of 94 and 33 rows for 32.  FP64, periodic /
// zero p, with the boundary rule between the loads of an edge -> with them in
// groups: 64^2 13 / 20 -> 7 / 7 us, 256^2 15 / 28 -> 8 / 8, 2048^2 21 / 44 -> 15
// / 14, 4096^2 59 / 79 -> 51 / 49.  No register spilled (206 to 242 in FP64, two
// waves per SIMD).  2048^2 with two transposes around a sweep of rows: 70 us.
constexpr int GS_RK = 32;
template <typename T, int BC, bool THROUGH>
static __global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void k_gs_cols(const T *__restrict__ fin, T *__restrict__ fout, int nx, int np, const double *__restrict__ F, double dt,
               double dp, const double *__restrict__ gcoef, int ntx, int nty)
{
    int tx, ty;
    if (!xcd_tile(ntx, nty, tx, ty)) return;
    const int i = min(tx * 64 + ((int)threadIdx.x & 63), nx - 1);  // lanes past the last column repeat it
    const int j0 = (ty * 4 + ((int)threadIdx.x >> 6)) * GS_RK;
    if (j0 >= np) return;
    const Foot ft = foot_of_shift((F[i] * dt) / dp);
    const int m = foot_offset<BC, FOOT_MARGIN_GS>(ft, np);
    const size_t ld = (size_t)nx;
    int q0 = j0 + m - GS_K - 1;  // row of sample 0
    if (BC == BC_PERIODIC) q0 = wrap_near(q0, np);
    const T r = (T)gcoef[0], cD = (T)gcoef[1], a = (T)ft.a, b = (T)ft.b, g = (T)ft.g, d = (T)ft.d;
    T y[GS_RK + GS_K];
    int o = 0;
    __asm__ __volatile__("" : "+v"(o));  // the second reads are reads
    if (__builtin_amdgcn_readfirstlane((int)__all(q0 >= 0 && q0 + GS_RK + 2 * GS_K + 2 <= np))) {
        // no sample of the wave needs the boundary rule
        const T *col = fin + (size_t)q0 * ld + i;
        gs_cells<GS_RK>(GsDirect<T>{col, ld}, GsDirect<T>{col + o, ld}, r, cD, a, b, g, d, y);
    } else {
        using Edge = GsEdge<T, BC, GS_RK + 1>;
        gs_cells<GS_RK>(Edge{fin + i, ld, q0, np}, Edge{fin + i, ld, q0 + o, np}, r, cD, a, b, g, d, y);
    }
#pragma unroll
    for (int u = 0; u < GS_RK; ++u)
        if (j0 + u < np) store1<THROUGH>(fout + (size_t)(j0 + u) * ld + i, y[u]);
}

// Density partial sums of f (serial over the rows of each 16-row block, in
// the order the drift kernels accumulate them).
template <typename T>
static __global__ __launch_bounds__(256) void k_partials(const T *__restrict__ f, double *__restrict__ part, int nx,
                                                  int np)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= nx) return;
    const int b = blockIdx.y;
    const int jend = min(b * ROWS_PER_BLOCK + ROWS_PER_BLOCK, np);
    double acc = 0.0;
    for (int j = b * ROWS_PER_BLOCK; j < jend; ++j) acc = acc + (double)f[(size_t)j * nx + i];
    part[(size_t)b * nx + i] = acc;
}

// ---------------------------------------------------------------------------
// Density rho_i = dp * sum_j f_ji from the 16-row partial sums.  One
// workgroup per 16 columns: thread (c, g) forms the serial sums of the block
// classes l = g, g + 16, g + 32, g + 48 (blocks b = l mod 64, ascending b) of
// column c, so that a wavefront load reads 16 adjacent columns of 4 block
// rows; the 64 class sums of a column are then combined by the pairwise tree
// in LDS.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void density_block(const double *__restrict__ part, double *__restrict__ rho, int nx,
                                              int nblk, double dp, int blk, double (*S)[17])
{
    const int c = threadIdx.x & 15;
    const int g = threadIdx.x >> 4;
    const int i = blk * 16 + c;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    if (i < nx) {
        for (int b0 = 0; b0 < nblk; b0 += 64) {
            double x[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int b = b0 + g + 16 * k;
                x[k] = b < nblk ? part[(size_t)b * nx + i] : 0.0;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (b0 + g + 16 * k < nblk) acc[k] = acc[k] + x[k];
        }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) S[g + 16 * k][c] = acc[k];
    __syncthreads();
    for (int d = 32; d >= 1; d >>= 1) {
        for (int k = threadIdx.x; k < d * 16; k += 256) {
            const int l = k >> 4, cc = k & 15;
            S[l][cc] = S[l][cc] + S[l + d][cc];
        }
        __syncthreads();
    }
    if (g == 0 && i < nx) rho[i] = dp * S[0][c];
}


// The same sums with 1024 threads: thread (c, g) forms the serial sum of
// block class g alone, its loads (blocks g, g + 64, g + 128, g + 192 of a
// round) all in flight at once; then wavefront c folds the 64 class sums of
// column c with the xor butterfly (the same association as the pairwise tree
// S[g] + S[g + d], d = 32, ..., 1: addition is commutative).
static __global__ __launch_bounds__(1024) void k_density(const double *__restrict__ part, double *__restrict__ rho,
                                                  int nx, int nblk, double dp)
{
    __shared__ double S[16][65];
    const int c = threadIdx.x & 15, g = threadIdx.x >> 4;
    const int i = blockIdx.x * 16 + c;
    const int ic = min(i, nx - 1);
    double acc = 0.0;
    for (int b0 = 0; b0 < nblk; b0 += 256) {
        double x[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            x[k] = part[(size_t)min(b0 + g + 64 * k, nblk - 1) * nx + ic];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) keep_issued(x[k]);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (b0 + g + 64 * k < nblk) acc = acc + x[k];
    }
    S[c][g] = acc;
    __syncthreads();
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const double v = wave_sum(S[w][lane]);
    const int io = blockIdx.x * 16 + w;
    if (lane == 0 && io < nx) rho[io] = dp * v;
}

// Stage two arrays of n doubles into LDS (whole workgroup), the sixteen loads
// of a round per thread in flight before their LDS writes.
__device__ __forceinline__ void stage2(double *d0, const double *__restrict__ s0, double *d1,
                                       const double *__restrict__ s1, int n)
{
    const int bd = blockDim.x;
    for (int k0 = threadIdx.x; k0 < n; k0 += 8 * bd) {
        double v[2][8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int k = min(k0 + u * bd, n - 1);
            v[0][u] = s0[k];
            v[1][u] = s1[k];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            keep_issued(v[0][u]);
            keep_issued(v[1][u]);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (k0 + u * bd < n) {
                d0[k0 + u * bd] = v[0][u];
                d1[k0 + u * bd] = v[1][u];
            }
    }
}

// Stage three arrays of n doubles into LDS (whole workgroup), the twelve
// loads of a round per thread in flight before their LDS writes.
__device__ __forceinline__ void stage3(double *d0, const double *__restrict__ s0, double *d1,
                                       const double *__restrict__ s1, double *d2, const double *__restrict__ s2, int n)
{
    const int bd = blockDim.x;
    for (int k0 = threadIdx.x; k0 < n; k0 += 4 * bd) {
        double v[3][4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int k = min(k0 + u * bd, n - 1);
            v[0][u] = s0[k];
            v[1][u] = s1[k];
            v[2][u] = s2[k];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            keep_issued(v[0][u]);
            keep_issued(v[1][u]);
            keep_issued(v[2][u]);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (k0 + u * bd < n) {
                d0[k0 + u * bd] = v[0][u];
                d1[k0 + u * bd] = v[1][u];
                d2[k0 + u * bd] = v[2][u];
            }
    }
}

// Magnetization of eq. (mxmydef) by one wavefront from LDS copies of rho, cos
// and sin; every lane returns (mx, my).
__device__ inline void magnetization(const double *rho, const double *cs, const double *sn, int n, double dx,
                                     double &mx, double &my)
{
    const int lane = threadIdx.x & 63;
    double c = 0.0, s = 0.0;
    int i = lane;
    // eight terms of each chain requested at once (the chains stay in order)
    for (; i + 7 * 64 < n; i += 8 * 64) {
        double cv[8], sv[8], rv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            cv[u] = cs[i + 64 * u];
            sv[u] = sn[i + 64 * u];
            rv[u] = rho[i + 64 * u];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            c = fma(cv[u], rv[u], c);
            s = fma(sv[u], rv[u], s);
        }
    }
    for (; i < n; i += 64) {
        c = fma(cs[i], rho[i], c);
        s = fma(sn[i], rho[i], s);
    }
    c = wave_sum(c);
    s = wave_sum(s);
    mx = dx * c;
    my = dx * s;
}

// Keeps (mx, my) of the latest force evaluation and appends it to the history.
__device__ inline void record_history(double *mxmy, double *hist, int64_t *hcount, int64_t hcap, double mx,
                                      double my)
{
    mxmy[0] = mx;
    mxmy[1] = my;
    if (hcap <= 0) return;
    const int64_t c = *hcount;
    if (c < hcap) {
        hist[2 * c] = mx;
        hist[2 * c + 1] = my;
    }
    *hcount = c + 1;
}

constexpr int FORCE_LDS_MAX = 4096;  // nx up to which rho, cos, sin are staged in LDS

// HMF force, eq. (hmfmeanforce): F_i = -sin(x_i) M_x + cos(x_i) M_y.  One
// workgroup; wavefront 0 forms (M_x, M_y).  L: 3 SMAX doubles (STAGED, n <= SMAX).
template <bool STAGED, int SMAX = FORCE_LDS_MAX>
__device__ __forceinline__ void force_hmf_block(const double *__restrict__ rho, const double *__restrict__ cs,
                                                const double *__restrict__ sn, double *__restrict__ F, int n,
                                                double dx, double *mxmy, double *hist, int64_t *hcount, int64_t hcap,
                                                double *L, double *M)
{
    const double *r = rho, *c = cs, *s = sn;
    if (STAGED) {
        stage3(L, rho, L + SMAX, cs, L + 2 * SMAX, sn, n);
        __syncthreads();
        r = L;
        c = L + SMAX;
        s = L + 2 * SMAX;
    }
    if (threadIdx.x < 64) {
        double mx, my;
        magnetization(r, c, s, n, dx, mx, my);
        if (threadIdx.x == 0) {
            M[0] = mx;
            M[1] = my;
            record_history(mxmy, hist, hcount, hcap, mx, my);
        }
    }
    __syncthreads();
    const double mx = M[0], my = M[1];
    for (int i = threadIdx.x; i < n; i += blockDim.x) F[i] = fma(my, c[i], -(mx * s[i]));
}

// The single-grid form: wavefront 0 forms (M_x, M_y) from the arrays in
// memory (the same chains as magnetization()), then every thread writes its
// forces; no staging of the three arrays.  One wavefront's chain bounds it.
// AHEAD (more columns than threads): the factors of a thread's first forces
// are requested before that chain, not after it (4096 columns 5.4 -> 4.4 us;
// with fewer columns the requests delay the chain: 128, a step 11.5 -> 11.6).
template <bool AHEAD>
static __global__ __launch_bounds__(1024) void k_force_hmf(const double *__restrict__ rho, const double *__restrict__ cs,
                                                    const double *__restrict__ sn, double *__restrict__ F, int n,
                                                    double dx, double *mxmy, double *hist, int64_t *hcount,
                                                    int64_t hcap)
{
    __shared__ double M[2];
    constexpr int U = AHEAD ? 4 : 0;
    double cv[U + 1], sv[U + 1];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int i = min((int)(threadIdx.x + u * blockDim.x), n - 1);
        cv[u] = cs[i];
        sv[u] = sn[i];
    }
    if (threadIdx.x < 64) {
        double mx, my;
        magnetization(rho, cs, sn, n, dx, mx, my);
        if (threadIdx.x == 0) {
            M[0] = mx;
            M[1] = my;
            record_history(mxmy, hist, hcount, hcap, mx, my);
        }
    }
    __syncthreads();
    const double mx = M[0], my = M[1];
    int i = threadIdx.x;
#pragma unroll
    for (int u = 0; u < U; ++u, i += blockDim.x)
        if (i < n) F[i] = fma(my, cv[u], -(mx * sv[u]));
    for (; i < n; i += blockDim.x) F[i] = fma(my, cs[i], -(mx * sn[i]));
}

// Magnetization only (ring model, batched force phase).  One workgroup,
// wavefront 0 reduces.  L: 3 SMAX doubles (STAGED, n <= SMAX).
template <bool STAGED, int SMAX = FORCE_LDS_MAX>
__device__ __forceinline__ void magnetization_block(const double *__restrict__ rho, const double *__restrict__ cs,
                                                    const double *__restrict__ sn, int n, double dx, double *mxmy,
                                                    double *hist, int64_t *hcount, int64_t hcap, double *L)
{
    const double *r = rho, *c = cs, *s = sn;
    if (STAGED) {
        stage3(L, rho, L + SMAX, cs, L + 2 * SMAX, sn, n);
        __syncthreads();
        r = L;
        c = L + SMAX;
        s = L + 2 * SMAX;
    }
    if (threadIdx.x < 64) {
        double mx, my;
        magnetization(r, c, s, n, dx, mx, my);
        if (threadIdx.x == 0) record_history(mxmy, hist, hcount, hcap, mx, my);
    }
}

// Ring force, eq. (meanforce) with eq. (ringpot): F_i = -dx sum_k K_{(i-k)
// mod n} rho_k with K the tabulated V'.  One wavefront per output i.
__device__ __forceinline__ void force_ring_output(const double *__restrict__ rho, const double *__restrict__ K,
                                                  double *__restrict__ F, int n, double dx, int i)
{
    const int lane = threadIdx.x & 63;
    double acc = 0.0;
    int k = lane;
    // eight terms of the chain requested at once (the chain stays in order)
    for (; k + 7 * 64 < n; k += 8 * 64) {
        double kv[8], rv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            int d = i - (k + 64 * u);
            if (d < 0) d += n;
            kv[u] = K[d];
            rv[u] = rho[k + 64 * u];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) acc = fma(kv[u], rv[u], acc);
    }
    for (; k < n; k += 64) {
        int d = i - k;
        if (d < 0) d += n;
        acc = fma(K[d], rho[k], acc);
    }
    acc = wave_sum(acc);
    if (lane == 0) F[i] = -(dx * acc);
}

// Four adjacent outputs i0 .. i0 + 3 by one wavefront, their chains side by
// side over the same density values.
__device__ __forceinline__ void force_ring_outputs4(const double *__restrict__ rho, const double *__restrict__ K,
                                                    double *__restrict__ F, int n, double dx, int i0)
{
    const int lane = threadIdx.x & 63;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int k0 = lane; k0 < n; k0 += 4 * 64) {
        double kv[4][4], rv[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int k = min(k0 + 64 * u, n - 1);
            rv[u] = rho[k];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int d = min(i0 + q, n - 1) - k;
                kv[u][q] = K[d < 0 ? d + n : d];
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            keep_issued(rv[u]);
#pragma unroll
            for (int q = 0; q < 4; ++q) keep_issued(kv[u][q]);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (k0 + 64 * u < n)
#pragma unroll
                for (int q = 0; q < 4; ++q) acc[q] = fma(kv[u][q], rv[u], acc[q]);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] = wave_sum(acc[q]);
    if (lane < 4 && i0 + lane < n) F[i0 + lane] = -(dx * (lane == 0 ? acc[0] : lane == 1 ? acc[1] : lane == 2 ? acc[2] : acc[3]));
}

// Workgroup 0 forms the magnetization (M_x, M_y) for the history instead (the
// ring force does not use it), dispatched first so that its chain overlaps
// the outputs' workgroups.  STAGED (n <= RING_LDS_MAX): every workgroup first
// copies the arrays it reads (rho and K; rho, cos and sin for workgroup 0)
// into LDS, whose reads in the chains are conflict-free (adjacent lanes,
// adjacent words), and its four wavefronts then form RING_OUT_WG / 4 outputs
// each; otherwise one output per wavefront straight from global memory.
// Launch 1 + ceil(n / ring_outputs_per_wg(n)) workgroups of 256 threads.
constexpr int RING_LDS_MAX = 2048;
constexpr int RING_OUT_WG = 8;
__host__ __device__ constexpr int ring_outputs_per_wg(int n) { return n <= RING_LDS_MAX ? RING_OUT_WG : 4; }

template <bool STAGED>
static __global__ __launch_bounds__(256) void k_force_ring(const double *__restrict__ rho, const double *__restrict__ K,
                                                    double *__restrict__ F, int n, double dx,
                                                    const double *__restrict__ cs, const double *__restrict__ sn,
                                                    double *mxmy, double *hist, int64_t *hcount, int64_t hcap)
{
    __shared__ double L[STAGED ? 3 * RING_LDS_MAX : 1];
    if (blockIdx.x == 0) {
        const double *r = rho, *c = cs, *s = sn;
        if (STAGED) {
            stage3(L, rho, L + RING_LDS_MAX, cs, L + 2 * RING_LDS_MAX, sn, n);
            __syncthreads();
            r = L;
            c = L + RING_LDS_MAX;
            s = L + 2 * RING_LDS_MAX;
        }
        if (threadIdx.x < 64) {
            double mx, my;
            magnetization(r, c, s, n, dx, mx, my);
            if (threadIdx.x == 0) record_history(mxmy, hist, hcount, hcap, mx, my);
        }
        return;
    }
    constexpr int OUT = STAGED ? RING_OUT_WG : 4;
    const double *r = rho, *k = K;
    if (STAGED) {
        stage2(L, rho, L + RING_LDS_MAX, K, n);
        __syncthreads();
        r = L;
        k = L + RING_LDS_MAX;
    }
#pragma unroll
    for (int q = 0; q < OUT / 4; ++q) {
        const int i = (blockIdx.x - 1) * OUT + (threadIdx.x >> 6) * (OUT / 4) + q;
        if (i < n) force_ring_output(r, k, F, n, dx, i);
    }
}

// Sheet force, eq. (sheetpot) with V = 2 pi G |x|: F_i = K (S - 2 P_i - rho_i),
// K = 2 pi G dx, P_i the exclusive prefix sum of rho and S its total.
// Wavefront 0 scans: lane l owns the contiguous chunk [l c, (l+1) c),
// c = ceil(n/64), and replaces each sample by the sum of those before it in
// the chunk; chunk totals by an inclusive Hillis-Steele scan d = 1, 2, ..., 32.
// P_i is the sum before the chunk (X[l], of X[65]; X[64] is S) plus that
// before i in it, and all threads form the forces.  When staged, the samples
// are held in LDS chunk-transposed (element l c + k at k 65 + l) so that the
// 64 lanes walking their chunks use adjacent words; else in F.  Bound by the
// one wavefront's chain of additions: with the forces in a second walk of that
// wavefront 4096 columns took 4.9 us, 4.2 now.
constexpr int SHEET_LDS_MAX = 16384;
constexpr int SHEET_LDS_WORDS = (SHEET_LDS_MAX / 64) * 65;

// The scan: samples replaced by the sums before them in their chunks, X as above.
template <bool STAGED>
__device__ __forceinline__ void sheet_scan(const double *__restrict__ rho, double *__restrict__ F, int n, int c,
                                           double *L, double *X)
{
    if (threadIdx.x < 64) {
        const int l = threadIdx.x;
        const int len = min(c, n - l * c);  // <= 0 past the end
        double tot = 0.0;
        // (past the chunk: any value in bounds, not used)
        auto at = [&](int k) { return STAGED ? L[min(k, c - 1) * 65 + l] : rho[min(l * c + k, n - 1)]; };
        auto one = [&](int k, double r) {
            if (STAGED)
                L[k * 65 + l] = tot;
            else
                F[l * c + k] = tot;
            tot = tot + r;
        };
        // eight samples ahead, summed in order
        constexpr int B = 8;
        double v[B], w[B];
#pragma unroll
        for (int u = 0; u < B; ++u) v[u] = at(u);
        int k = 0;
        for (; k + B <= len; k += B) {
#pragma unroll
            for (int u = 0; u < B; ++u) w[u] = at(k + B + u);
#pragma unroll
            for (int u = 0; u < B; ++u) one(k + u, v[u]);
#pragma unroll
            for (int u = 0; u < B; ++u) v[u] = w[u];
        }
#pragma unroll
        for (int u = 0; u < B; ++u)
            if (k + u < len) one(k + u, v[u]);
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const double up = __shfl_up(tot, d, 64);
            if (l >= d) tot = up + tot;
        }
        X[l + 1] = tot;
        if (l == 0) X[0] = 0.0;
    }
    __syncthreads();
}

template <bool STAGED>
__device__ __forceinline__ void force_sheet_block(const double *__restrict__ rho, double *__restrict__ F, int n,
                                                  double K, double *L, double *X)
{
    const int c = (n + 63) / 64;
    const int bd = blockDim.x;
    // i / c: for n <= SHEET_LDS_MAX (c <= 256) the float product is off by less
    // than 1e-4 where its distance from a whole number is at least 1 / (2 c)
    const float rc = 1.0f / (float)c;
    auto chunk = [&](int i) { return STAGED ? (int)(((float)i + 0.5f) * rc) : i / c; };
    constexpr int U = 4;  // samples of a thread requested together
    double own[U];        // the first ones stay in registers for the result
    if (STAGED) {
        for (int i0 = threadIdx.x; i0 < n; i0 += U * bd) {
            double v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = rho[min(i0 + u * bd, n - 1)];
#pragma unroll
            for (int u = 0; u < U; ++u) keep_issued(v[u]);
            if (i0 == (int)threadIdx.x)
#pragma unroll
                for (int u = 0; u < U; ++u) own[u] = v[u];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = i0 + u * bd, l = chunk(i);
                if (i < n) L[(i - l * c) * 65 + l] = v[u];
            }
        }
        __syncthreads();
    }
    sheet_scan<STAGED>(rho, F, n, c, L, X);
    const double S = X[64];
    auto force = [&](int i, double r) {
        const int l = chunk(i);
        const double Pi = X[l] + (STAGED ? L[(i - l * c) * 65 + l] : F[i]);
        F[i] = K * (fma(-2.0, Pi, S) - r);
    };
    int i = threadIdx.x;
    if (STAGED) {
#pragma unroll
        for (int u = 0; u < U; ++u, i += bd)
            if (i < n) force(i, own[u]);
    }
    for (; i < n; i += bd) force(i, rho[i]);
}

template <bool STAGED>
static __global__ __launch_bounds__(1024) void k_force_sheet(const double *__restrict__ rho, double *__restrict__ F, int n,
                                                      double K)
{
    __shared__ double L[STAGED ? SHEET_LDS_WORDS : 1];
    __shared__ double X[65];
    force_sheet_block<STAGED>(rho, F, n, K, L, X);
}

// Density and force of a small grid in one launch, for HMF (model 0) and sheet
// (model 2) by one workgroup, a thread per column.  The two kernels take a launch
// and a few dependent memory latencies each, whatever the size: apart 3.9 us at
// 64^2, 4.4 at 128^2, 4.7 at 256^2 and 512^2 (HMF), together 2.0, 2.1, 2.5 and
// 4.1.  At 512^2 reading the partial sums through one CU (64 KB in 1 us) takes
// up most of what the launch saves; hence SMALL_PART.  A column's classes are
// of one block each (at most 32), summed by the butterfly's tree in the
// thread's registers; classes past the last block are 0.
constexpr int SMALL_NX = 1024, SMALL_BLK = 32, SMALL_PART = 16384;
__host__ __device__ constexpr bool small_grid(int64_t nx, int64_t nblk)
{
    return nx <= SMALL_NX && nblk <= SMALL_BLK && nx * nblk <= SMALL_PART;
}

template <int NB>
__device__ __forceinline__ double column_sum(const double *__restrict__ part, int i, int nx, int nblk)
{
    double v[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) v[b] = part[(size_t)min(b, nblk - 1) * nx + i];
#pragma unroll
    for (int b = 0; b < NB; ++b) keep_issued(v[b]);
    // 0 + x: the classes' sums start from 0
#pragma unroll
    for (int b = 0; b < NB; ++b) v[b] = b < nblk ? 0.0 + v[b] : 0.0;
#pragma unroll
    for (int d = NB / 2; d >= 1; d >>= 1)
#pragma unroll
        for (int b = 0; b < d; ++b) v[b] = v[b] + v[b + d];
    return v[0];
}

__device__ __forceinline__ double column_density(const double *__restrict__ part, int i, int nx, int nblk, double dp)
{
    return dp * (nblk <= 8    ? column_sum<8>(part, i, nx, nblk)
                 : nblk <= 16 ? column_sum<16>(part, i, nx, nblk)
                              : column_sum<SMALL_BLK>(part, i, nx, nblk));
}

// The ring's form: the workgroups of k_force_ring<true>, each of which sums all
// columns for itself (they are few, and come from the caches); workgroup 0
// keeps the densities.  A step, in two launches -> one: 64^2 13.6 -> 9.7 us,
// 256^2 14.6 -> 10.8, 512^2 14.3 -> 12.8, 1024 x 256 14.9 -> 13.4.
static __global__ __launch_bounds__(256) void k_density_force_ring(
    const double *__restrict__ part, double *__restrict__ rho, const double *__restrict__ K, double *__restrict__ F,
    int n, int nblk, double dp, double dx, const double *__restrict__ cs, const double *__restrict__ sn, double *mxmy,
    double *hist, int64_t *hcount, int64_t hcap)
{
    constexpr int U = SMALL_NX / 256;
    __shared__ double L[3 * SMALL_NX];
    const bool mag = blockIdx.x == 0;
    const int t = threadIdx.x;
    const double *a0 = mag ? cs : K;  // staged beside the densities
    double v0[U], v1[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int i = min(t + 256 * u, n - 1);
        v0[u] = a0[i];
        v1[u] = sn[i];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int i = t + 256 * u;
        if (256 * u >= n) break;  // uniform
        const double r = column_density(part, min(i, n - 1), n, nblk, dp);
        L[i] = r;
        L[SMALL_NX + i] = v0[u];
        L[2 * SMALL_NX + i] = v1[u];
        if (mag && i < n) rho[i] = r;
    }
    __syncthreads();
    if (mag) {
        if (t < 64) {
            double mx, my;
            magnetization(L, L + SMALL_NX, L + 2 * SMALL_NX, n, dx, mx, my);
            if (t == 0) record_history(mxmy, hist, hcount, hcap, mx, my);
        }
        return;
    }
#pragma unroll
    for (int q = 0; q < RING_OUT_WG / 4; ++q) {
        const int i = (blockIdx.x - 1) * RING_OUT_WG + (t >> 6) * (RING_OUT_WG / 4) + q;
        if (i < n) force_ring_output(L, L + SMALL_NX, F, n, dx, i);
    }
}

template <int MODEL>
static __global__ __launch_bounds__(SMALL_NX) void k_density_force(
    const double *__restrict__ part, double *__restrict__ rho, double *__restrict__ F, int n, int nblk, double dp,
    const double *__restrict__ cs, const double *__restrict__ sn, double dx, double *mxmy, double *hist,
    int64_t *hcount, int64_t hcap, double K)
{
    __shared__ double L[3 * SMALL_NX];
    __shared__ double X[65];
    const int i = threadIdx.x, ic = min(i, n - 1);
    double cv = 0.0, sv = 0.0;
    if (MODEL == 0) {
        cv = cs[ic];
        sv = sn[ic];
    }
    const double r = column_density(part, ic, n, nblk, dp);
    if (i < n) rho[i] = r;
    if (MODEL == 0) {
        L[i] = r;
        L[SMALL_NX + i] = cv;
        L[2 * SMALL_NX + i] = sv;
        __syncthreads();
        if (i < 64) {
            double mx, my;
            magnetization(L, L + SMALL_NX, L + 2 * SMALL_NX, n, dx, mx, my);
            if (i == 0) {
                X[0] = mx;
                X[1] = my;
                record_history(mxmy, hist, hcount, hcap, mx, my);
            }
        }
        __syncthreads();
        if (i < n) F[i] = fma(X[1], cv, -(X[0] * sv));
    } else {
        const int c = (n + 63) / 64;
        const int l = ic / c, slot = (ic - l * c) * 65 + l;
        if (i < n) L[slot] = r;
        __syncthreads();
        sheet_scan<true>(rho, F, n, c, L, X);
        if (i < n) F[i] = K * (fma(-2.0, X[l] + L[slot], X[64]) - r);
    }
}

// ---------------------------------------------------------------------------
// Diagnostics.  Pass 1: 16-row block sums of f, p f, p^2/2 f and f^2 (SETS bit
// 0) and of f log f over f > 0 (entropy density) and f over f < 0 (negative
// mass; bit 1), one plane of the scratch each.  One thread per column and
// block, its sixteen rows requested together.  Both sets in one pass read f
// once (2048^2 FP64: 8.4 + 16.2 us apart, 17.5 together, of which most is the
// log).
// ---------------------------------------------------------------------------
template <typename T, int SETS>
static __global__ __launch_bounds__(256) void k_mom_blocks(const T *__restrict__ f, double *__restrict__ scratch, int nx,
                                                    int np, int nblk, double pmin, double dp)
{
    constexpr int R = ROWS_PER_BLOCK;
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= nx) return;
    const int b = blockIdx.y;
    const int j0 = b * R;
    const int nr = min(R, np - j0);
    T x[R];
#pragma unroll
    for (int r = 0; r < R; ++r) x[r] = f[(size_t)(j0 + min(r, nr - 1)) * nx + i];
#pragma unroll
    for (int r = 0; r < R; ++r) keep_issued(x[r]);
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0, se = 0.0, sn = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (r < nr) {  // uniform
            const double v = (double)x[r];
            if (SETS & 1) {
                const double pj = pmin + (double)(j0 + r) * dp;
                const double kj = 0.5 * (pj * pj);
                s0 = s0 + v;
                s1 = fma(pj, v, s1);
                s2 = fma(kj, v, s2);
                s3 = fma(v, v, s3);
            }
            if (SETS & 2) {
                se = se + (v > 0.0 ? v * log(v) : 0.0);
                sn = sn + (v < 0.0 ? v : 0.0);
            }
        }
    }
    const size_t plane = (size_t)nblk * nx;
    double *o = scratch + (size_t)b * nx + i;
    if (SETS & 1) {
        o[0] = s0;
        o[plane] = s1;
        o[2 * plane] = s2;
        o[3 * plane] = s3;
        o += 4 * plane;
    }
    if (SETS & 2) {
        o[0] = se;
        o[plane] = sn;
    }
}

// Pass 2: column quantities col[q0 + q][i] = dp * sum over blocks of scratch
// plane q < NQ: the sums of k_density for NQ planes, the loads of all planes in
// flight together (2048^2, six planes: 7.2 us; 13 with a wavefront reading down
// each column).
template <int NQ>
static __global__ __launch_bounds__(1024) void k_mom_cols(const double *__restrict__ scratch, double *__restrict__ col,
                                                   int nx, int nblk, double dp, int q0)
{
    __shared__ double S[NQ][16][65];
    const int c = threadIdx.x & 15, g = threadIdx.x >> 4;
    const int ic = min((int)blockIdx.x * 16 + c, nx - 1);
    const size_t plane = (size_t)nblk * nx;
    double acc[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc[q] = 0.0;
    for (int b0 = 0; b0 < nblk; b0 += 128) {
        double x[NQ][2];
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int k = 0; k < 2; ++k) x[q][k] = scratch[q * plane + (size_t)min(b0 + g + 64 * k, nblk - 1) * nx + ic];
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int k = 0; k < 2; ++k) keep_issued(x[q][k]);
#pragma unroll
        for (int k = 0; k < 2; ++k)
            if (b0 + g + 64 * k < nblk)
#pragma unroll
                for (int q = 0; q < NQ; ++q) acc[q] = acc[q] + x[q][k];
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) S[q][c][g] = acc[q];
    __syncthreads();
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int io = blockIdx.x * 16 + w;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const double v = wave_sum(S[q][w][lane]);
        if (lane == 0 && io < nx) col[(size_t)(q0 + q) * nx + io] = dp * v;
    }
}

// Pass 3 (ring and sheet): phi_i = sum_k V(x_i - x_k) rho_k with V the
// tabulated ring potential, or |i - k| (sheet, in cells).  One wavefront per
// output, eight terms of its chain requested at once.
template <bool RING>
static __global__ __launch_bounds__(256) void k_mom_phi(const double *__restrict__ rho, const double *__restrict__ V,
                                                 double *__restrict__ phi, int n)
{
    const int lane = threadIdx.x & 63;
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= n) return;
    double acc = 0.0;
    for (int k0 = lane; k0 < n; k0 += 8 * 64) {
        double v[8], r[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int k = min(k0 + 64 * u, n - 1);
            const int d = i - k;
            v[u] = RING ? V[d < 0 ? d + n : d] : (double)(d < 0 ? -d : d);
            r[u] = rho[k];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) keep_issued(r[u]);
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (k0 + 64 * u < n) acc = fma(v[u], r[u], acc);
    }
    acc = wave_sum(acc);
    if (lane == 0) phi[i] = acc;
}

// Pass 4: totals, out = {mass, momentum, kinetic, potential, energy, mx, my,
// l2, entropy, negative mass}.  One wavefront per sum, sixteen terms of its
// chain requested at once (2048 columns: 4.9 us; 14 with all nine sums in one
// wavefront).
static __global__ __launch_bounds__(576) void k_mom_final(const double *__restrict__ col, const double *__restrict__ phi,
                                                   const double *__restrict__ cs, const double *__restrict__ sn,
                                                   double *__restrict__ out, int n, double dx, int model,
                                                   double wcoef)
{
    __shared__ double S[9];
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    const bool angular = (model == 0 || model == 1);
    const bool pair = (model == 1 || model == 2);
    // sums 0..5: the column quantities; 6, 7, 8: cos, sin and phi times rho
    const double *a = q < 6 ? col + (size_t)q * n : col;
    const double *b = q == 6 ? cs : (q == 7 ? sn : phi);
    double s = 0.0;
    if (q < 6 || (q < 8 ? angular : pair)) {
        for (int k0 = lane; k0 < n; k0 += 16 * 64) {
            double x[16], y[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int k = min(k0 + 64 * u, n - 1);
                x[u] = a[k];
                y[u] = q < 6 ? 0.0 : b[k];
            }
#pragma unroll
            for (int u = 0; u < 16; ++u) keep_issued(x[u]);
#pragma unroll
            for (int u = 0; u < 16; ++u)
                if (k0 + 64 * u < n) s = q < 6 ? s + x[u] : fma(y[u], x[u], s);
        }
        s = wave_sum(s);
    }
    if (lane == 0) S[q] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        const double mass = dx * S[0], kin = dx * S[2];
        double mx = 0.0, my = 0.0, W = 0.0;
        if (angular) {
            mx = dx * S[6];
            my = dx * S[7];
        }
        if (model == 0)
            W = 0.5 * ((mass * mass - mx * mx) - my * my);
        else if (pair)
            W = wcoef * S[8];
        out[0] = mass;
        out[1] = dx * S[1];
        out[2] = kin;
        out[3] = W;
        out[4] = kin + W;
        out[5] = mx;
        out[6] = my;
        out[7] = dx * S[3];
        out[8] = -(dx * S[4]);
        out[9] = dx * S[5];
    }
}

// ---------------------------------------------------------------------------
// Batches: many grids (of one storage type) stepped together, one persistent
// launch per phase.  A grid is described by a GridDesc; a cycle (drift,
// density, force, kick) by a Cycle listing the member grids, what each does in
// that cycle and the prefix offsets of their work items.  Workgroups stride
// over the work items of all members; per-grid arithmetic is exactly that of
// the single-grid kernels, whatever workgroup processes a tile.
// ---------------------------------------------------------------------------
// The counts of members and work items are arguments where the launch knows
// them (items >= 0; two dependent loads fewer before the first item), else
// (a captured launch) read from the table.
constexpr int BATCH_MAX = 256;

enum { DRIFT_NONE = 0, DRIFT_FIRST = 1, DRIFT_PAIR = 2, DRIFT_LAST = 3 };
// no kick, a separate one, one fused with the two half drifts after it, or (last
// step) with the one after it
enum { KICK_NONE = 0, KICK_ALONE = 1, KICK_PAIR = 2, KICK_LAST = 3 };

struct GridDesc {
    void *f[2];
    const int32_t *dm;
    const double4 *dw;
    double *part, *rho, *F;
    const double *Fkick;  // force read by the kick (F, or the EXTERNAL table)
    const double *cs, *sn, *K;
    double *mxmy, *hist;
    int64_t *hcount;
    int64_t hcap;
    int32_t nx, np, nblk, model, bc_x, bc_p;
    int32_t kd_wide;  // fused kick and drift on the wide-slack tiles
    double dx, dp, dt, sheetK;
    const int32_t *kbase, *krel;  // fused kick and drift: tables of the member's 16-row tiles
};

struct Cycle {
    int32_t n;                   // members in this cycle (member a has GridDesc a)
    int8_t drift[BATCH_MAX];     // DRIFT_* (FIRST and PAIR also write density partial sums)
    int8_t kick[BATCH_MAX];      // KICK_* (all but NONE with density and force)
    int8_t cur[BATCH_MAX];       // current f buffer at the start of the cycle
    int8_t kin[BATCH_MAX];       // f buffer the kick (or fused kick and drift) reads
    int8_t pad[4];
    // work items of the phases: drift tiles, density blocks, force items,
    // tiles of the separate kick, tiles of the fused kick and two half drifts
    int32_t off_drift[BATCH_MAX + 1], off_dens[BATCH_MAX + 1], off_force[BATCH_MAX + 1], off_kick[BATCH_MAX + 1],
        off_kd[BATCH_MAX + 1];
};

// Member owning work item e: the last a with off[a] <= e (off[0] = 0 <= e <
// off[n]).  The lanes of each wavefront look at 64 members at a time: one
// memory latency, where a binary search had one per halving.
__device__ __forceinline__ int find_member(const int32_t *__restrict__ off, int n, int e)
{
    const int lane = threadIdx.x & 63;
    int count = 0;
    for (int base = 0; base < n; base += 64) {
        const int a = base + lane;
        const bool below = a < n && off[min(a, n)] <= e;
        count += __popcll(__ballot(below));
    }
    return count - 1;
}

// threadIdx.x, in FP64 anew for every work item: what the tiles of all kinds
// derive from it was computed before the loop over the items and spilled there
// (18 registers of the fused kernel, 10 of the drift).  Spilled -> not, FP64: 32
// grids of up to 1024 columns 3300 -> 2800 us, 8 of 2048^2 9420 -> 8450, one of
// 256^2 1170 -> 1075.  FP32 fits without.
template <typename T>
__device__ __forceinline__ int thread_of_item()
{
    int t = (int)threadIdx.x;
    if constexpr (sizeof(T) == 8) __asm__ __volatile__("" : "+v"(t));
    return t;
}

template <typename T>
static __global__ __launch_bounds__(KDGeom<DR_TW>::NT) __attribute__((amdgpu_waves_per_eu(8)))
void kb_drift(const GridDesc *__restrict__ gd, const Cycle *__restrict__ cy, int members, int items)
{
    using G = KDGeom<DR_TW>;
    __shared__ __attribute__((aligned(16))) T kbuf[G::NBUF * G::ROWLD];
    __shared__ __attribute__((aligned(16))) T mbuf[G::NBUF * G::ROWLD];
    __shared__ __attribute__((aligned(16))) T wtab[8 * ROWS_PER_BLOCK];
    const int n = items >= 0 ? members : cy->n;
    const int total = items >= 0 ? items : cy->off_drift[n];
    for (int e = blockIdx.x; e < total; e += gridDim.x) {
        const int a = find_member(cy->off_drift, n, e);
        const GridDesc &g = gd[a];
        const int kind = cy->drift[a], cur = cy->cur[a];
        const int li = e - cy->off_drift[a];
        const int ntx = (g.nx + DR_TW - 1) / DR_TW;
        __syncthreads();  // the previous item's LDS rows are consumed
        const int tid = thread_of_item<T>();
        const KDTile<T> t{(const T *)g.f[cur], (T *)g.f[cur ^ 1], nullptr, 0.0, 0.0, g.dm, g.dm, g.dw, g.dw, nullptr,
                          nullptr, kind == DRIFT_LAST ? nullptr : g.part, g.nx, g.np, 1, li % ntx, li / ntx, kbuf, mbuf,
                          wtab};
        if (g.bc_x == BC_PERIODIC) {
            if (kind == DRIFT_PAIR)
                kick_drift_tile<T, BC_PERIODIC, BC_PERIODIC, DR_TW, KD_SPR, 2, KD_LOAD, 2>(t, e, tid);
            else
                kick_drift_tile<T, BC_PERIODIC, BC_PERIODIC, DR_TW, KD_SPR, 2, KD_LOAD, 1>(t, e, tid);
        } else {
            if (kind == DRIFT_PAIR)
                kick_drift_tile<T, BC_ZERO, BC_PERIODIC, DR_TW, KD_SPR, 2, KD_LOAD, 2>(t, e, tid);
            else
                kick_drift_tile<T, BC_ZERO, BC_PERIODIC, DR_TW, KD_SPR, 2, KD_LOAD, 1>(t, e, tid);
        }
    }
}

static __global__ __launch_bounds__(256) void kb_density(const GridDesc *__restrict__ gd, const Cycle *__restrict__ cy, int members, int items)
{
    __shared__ double S[64][17];
    const int n = items >= 0 ? members : cy->n;
    const int total = items >= 0 ? items : cy->off_dens[n];
    for (int e = blockIdx.x; e < total; e += gridDim.x) {
        const int a = find_member(cy->off_dens, n, e);
        const GridDesc &g = gd[a];
        __syncthreads();
        density_block(g.part, g.rho, g.nx, g.nblk, g.dp, e - cy->off_dens[a], S);
    }
}

// Work items per member: HMF and sheet one workgroup; ring ceil(nx/16)
// workgroups of 16 outputs, four a wavefront, plus one for the magnetization;
// EXTERNAL none.  Arrays of the others are staged in LDS for grids up to
// BATCH_FORCE_STAGE columns.  Workgroups of four wavefronts: with sixteen (one
// ring output each) dispatching them took longer than the work (32 grids of up
// to 1024 columns: 9.2 us, 7.8 now).
constexpr int BATCH_FORCE_STAGE = 2048;
constexpr int BATCH_SHEET_WORDS = ((BATCH_FORCE_STAGE + 63) / 64) * 65;
constexpr int BATCH_FORCE_LDS = BATCH_SHEET_WORDS > 3 * BATCH_FORCE_STAGE ? BATCH_SHEET_WORDS : 3 * BATCH_FORCE_STAGE;

static __global__ __launch_bounds__(256) void kb_force(const GridDesc *__restrict__ gd, const Cycle *__restrict__ cy, int members, int items)
{
    __shared__ double L[BATCH_FORCE_LDS];
    __shared__ double M[65];
    const int n = items >= 0 ? members : cy->n;
    const int total = items >= 0 ? items : cy->off_force[n];
    for (int e = blockIdx.x; e < total; e += gridDim.x) {
        const int a = find_member(cy->off_force, n, e);
        const GridDesc &g = gd[a];
        const int li = e - cy->off_force[a];
        __syncthreads();
        if (g.model == 0) {
            if (g.nx <= BATCH_FORCE_STAGE)
                force_hmf_block<true, BATCH_FORCE_STAGE>(g.rho, g.cs, g.sn, g.F, g.nx, g.dx, g.mxmy, g.hist,
                                                         g.hcount, g.hcap, L, M);
            else
                force_hmf_block<false>(g.rho, g.cs, g.sn, g.F, g.nx, g.dx, g.mxmy, g.hist, g.hcount, g.hcap, L, M);
        } else if (g.model == 2) {
            if (g.nx <= BATCH_FORCE_STAGE)
                force_sheet_block<true>(g.rho, g.F, g.nx, g.sheetK, L, M);
            else
                force_sheet_block<false>(g.rho, g.F, g.nx, g.sheetK, L, M);
        } else if (g.model == 1) {
            const int nb = (g.nx + 15) / 16;
            if (li < nb) {
                force_ring_outputs4(g.rho, g.K, g.F, g.nx, g.dx, li * 16 + (threadIdx.x >> 6) * 4);
            } else if (g.nx <= BATCH_FORCE_STAGE) {
                magnetization_block<true, BATCH_FORCE_STAGE>(g.rho, g.cs, g.sn, g.nx, g.dx, g.mxmy, g.hist, g.hcount,
                                                             g.hcap, L);
            } else {
                magnetization_block<false>(g.rho, g.cs, g.sn, g.nx, g.dx, g.mxmy, g.hist, g.hcount, g.hcap, L);
            }
        }
    }
}

template <typename T, int R>
static __global__ __launch_bounds__(256) void kb_kick(const GridDesc *__restrict__ gd, const Cycle *__restrict__ cy, int members, int items)
{
    const int n = items >= 0 ? members : cy->n;
    const int total = items >= 0 ? items : cy->off_kick[n];
    for (int e = blockIdx.x; e < total; e += gridDim.x) {
        const int a = find_member(cy->off_kick, n, e);
        const GridDesc &g = gd[a];
        const int li = e - cy->off_kick[a];
        const int ntx = (g.nx + 255) / 256;
        const int tx = li % ntx, ty = li / ntx;
        const int kin = cy->kin[a];
        const T *fin = (const T *)g.f[kin];
        T *fout = (T *)g.f[kin ^ 1];
        if (g.bc_p == BC_PERIODIC)
            kick_tile<T, BC_PERIODIC, R>(fin, fout, g.Fkick, g.dt, g.dp, g.nx, g.np, tx, ty);
        else
            kick_tile<T, BC_ZERO, R>(fin, fout, g.Fkick, g.dt, g.dp, g.nx, g.np, tx, ty);
    }
}

// The kick fused with the two half drifts after it (the second of one step,
// the first of the next; only the former after the last kick) for the members
// whose tables allow it: tiles of 230
// columns by 16 rows with 8 columns of slack, as the single-grid kernel, or,
// for a member whose drift offsets spread more inside a tile (coarse p, fine
// x, long steps), tiles of 182 columns with 56 of slack (the same 256 kicked
// columns and four waves, more kicked columns per output).  Periodic p only.
constexpr int KB_KD_TW = 230;
// Rows requested ahead: with four, FP64 spills two registers (batches of up to
// 256 columns 1 to 3 % slower, of 2048^2 1 % faster).
constexpr int KB_PF = 2;
template <typename T>
static __global__ __launch_bounds__(KDGeom<KB_KD_TW>::NT) __attribute__((amdgpu_waves_per_eu(8)))
void kb_kick_drift(const GridDesc *__restrict__ gd, const Cycle *__restrict__ cy, int members, int items)
{
    using G = KDGeom<KB_KD_TW>;
    using GW = KDGeom<KD_TW_WIDE, KD_SPR_WIDE>;
    static_assert(G::NT == GW::NT && G::WK == GW::WK && G::W1 == GW::W1 && G::W2 == GW::W2 && G::ROWLD == GW::ROWLD &&
                      G::NBUF == GW::NBUF,
                  "one workgroup shape and wave roles for both tile widths");
    __shared__ __attribute__((aligned(16))) T kbuf[G::NBUF * G::ROWLD];
    __shared__ __attribute__((aligned(16))) T mbuf[G::NBUF * G::ROWLD];
    __shared__ __attribute__((aligned(16))) T wtab[8 * ROWS_PER_BLOCK];
    const int n = items >= 0 ? members : cy->n;
    const int total = items >= 0 ? items : cy->off_kd[n];
    for (int e = blockIdx.x; e < total; e += gridDim.x) {
        const int a = find_member(cy->off_kd, n, e);
        const GridDesc &g = gd[a];
        const int li = e - cy->off_kd[a];
        const int tw = g.kd_wide ? KD_TW_WIDE : KB_KD_TW;
        const int ntx = (g.nx + tw - 1) / tw;
        const int tx = li % ntx, ty = li / ntx;
        const int kin = cy->kin[a];
        const T *fin = (const T *)g.f[kin];
        T *fout = (T *)g.f[kin ^ 1];
        __syncthreads();  // the previous item's LDS rows are consumed
        const int tid = thread_of_item<T>();
        KDTile<T> t{fin, fout, g.Fkick, g.dt, g.dp, g.dm, g.dm, g.dw, g.dw, g.kbase, g.krel, g.part, g.nx, g.np, 1, tx, ty,
                          kbuf, mbuf, wtab};
        const bool px = g.bc_x == BC_PERIODIC;
#define KB_KD(TW, SPR)                                                                         \
    if (cy->kick[a] == KICK_LAST) {                                                            \
        t.part = nullptr;                                                                      \
        if (px)                                                                                \
            kick_drift_tile<T, BC_PERIODIC, BC_PERIODIC, TW, SPR, KB_PF, KD_KICK, 1>(t, e, tid); \
        else                                                                                   \
            kick_drift_tile<T, BC_ZERO, BC_PERIODIC, TW, SPR, KB_PF, KD_KICK, 1>(t, e, tid);     \
    } else if (px) {                                                                           \
        kick_drift_tile<T, BC_PERIODIC, BC_PERIODIC, TW, SPR, KB_PF, KD_KICK, 2>(t, e, tid);     \
    } else {                                                                                   \
        kick_drift_tile<T, BC_ZERO, BC_PERIODIC, TW, SPR, KB_PF, KD_KICK, 2>(t, e, tid);         \
    }
        if (g.kd_wide) {
            KB_KD(KD_TW_WIDE, KD_SPR_WIDE)
        } else {
            KB_KD(KB_KD_TW, KD_SPR)
        }
#undef KB_KD
    }
}

// Streaming copy (bandwidth ceiling): one 16-byte vector per thread, one
// 4 KiB tile per workgroup (the fastest of the copy shapes measured on the
// chip for buffers larger than its last-level cache).
static __global__ __launch_bounds__(256) void k_copy(const double2 *__restrict__ src, double2 *__restrict__ dst, size_t n)
{
    const size_t k = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (k < n) dst[k] = src[k];
}

}  // namespace vk
