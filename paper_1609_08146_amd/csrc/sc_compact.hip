// sc_compact.hip -- the compacted tables of a mirror's sum (see sc_compact.h), on the FP64 matrix
// instructions: c~ = (trigonometric interpolation)^T (Chebyshev interpolation)^T c per frequency.
//
//  k_compact_geometry   interpolation weights and the compacted nodes' records
//  k_compact_rows       T[m][phi] = sum_i L_m(theta_i) c[i][phi]        (contraction over the radii)
//  k_compact_cols       c~[m][p]  = sum_j D_m(phi_j - psi_p) T[m][phi_j] (contraction over phi)
//
// A record is four complex numbers (J~, rho~), 8 reals, so both steps are real matrix products with
// the 8 reals among their columns; v_mfma_f64_16x16x4 takes A[16][4] with lane l holding row l % 16,
// column l / 16, B[4][16] with row l / 16, column l % 16, and returns D[4 v + l / 16][l % 16].
// Everything is formed and summed in FP64, also for the FP32 form, whose compacted records are
// rounded to FP32 once at the end.
#include "sc_compact.h"
#include "sc_device.h"
#include "sc_internal.h"

namespace sc {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ double cheb_point(int j, int n) { return cospi((double)(2 * j + 1) / (double)(2 * n)); }

// Blocks of 64: first one per radius (radial weights), then the angular weights (one block per (16
// columns of a row, 64 phi)), then the compacted nodes.  Latency of a few sines each: 1.1e6 angular
// weights (400 phi, 2 700 nodes) took 67 us with one block for all phi of 16 columns.
constexpr int GEOM_PHI = 64;
__global__ void __launch_bounds__(64)
k_compact_geometry(CompactPlan plan, int n_r, int n_phi, double f, const double *__restrict__ r,
                   double *__restrict__ wrad, double *__restrict__ wang, double *__restrict__ pos64,
                   double *__restrict__ hinv64, float *__restrict__ pos32, float *__restrict__ dir32)
{
    const int lane = threadIdx.x, rows = plan.rows, rp = (rows + 15) / 16 * 16;
    const int n_i = (n_r + 4) / 4 * 4, n_g = (n_phi + GEOM_PHI - 1) / GEOM_PHI, n_a = plan.poff[rows] / 16 * n_g;
    int b = blockIdx.x;
    if (b < n_i) {
        // barycentric weights of the Chebyshev points: w_j = (-1)^j sin((2j + 1) pi / 2N)
        const double x = b <= n_r ? 4.0 * atan(r[b] / (2.0 * f)) / plan.theta_max - 1.0 : 0.0;
        double sum = 0.0;
        int hit = -1;
        for (int j = lane; j < rows; j += 64) {
            const double d = x - cheb_point(j, rows);
            if (d == 0.0) hit = j;
            const double w = sinpi((double)(2 * j + 1) / (double)(2 * rows));
            sum += (d == 0.0 ? 0.0 : ((j & 1) ? -w : w) / d);
        }
        for (int o = 32; o > 0; o >>= 1) {
            sum += __shfl_xor(sum, o);
            hit = max(hit, __shfl_xor(hit, o));
        }
        for (int j = lane; j < rp; j += 64) {
            double l = 0.0;
            if (b <= n_r && j < rows) {
                const double d = x - cheb_point(j, rows);
                const double w = sinpi((double)(2 * j + 1) / (double)(2 * rows));
                l = hit >= 0 ? (j == hit ? 1.0 : 0.0) : ((j & 1) ? -w : w) / d / sum;
            }
            wrad[(size_t)b * rp + j] = l;
        }
        return;
    }
    b -= n_i;
    if (b < n_a) {
        const int pt = b / n_g, j0 = (b - pt * n_g) * GEOM_PHI, j1 = min(j0 + GEOM_PHI, n_phi);
        int m = 0;
        while (plan.poff[m + 1] <= 16 * pt) ++m;
        const int P = plan.cols[m], p0 = 16 * pt - plan.poff[m], pp = (P + 15) / 16 * 16;
        double *w = wang + (size_t)plan.poff[m] * n_phi;
        const int p = p0 + (lane & 15);
        for (int j = j0 + (lane >> 4); j < j1; j += 4) {
            double d = 0.0;
            if (p < P) {
                // sin(P x / 2) / (P sin(x / 2)) at x = 2 pi (j / n_phi - p / P), on exact integers
                const int64_t a = (int64_t)j * P - (int64_t)p * n_phi;
                if (a == 0) d = 1.0;
                else if (P < n_phi)
                    d = sinpi((double)(a % (2 * (int64_t)n_phi)) / (double)n_phi) /
                        (P * sinpi((double)a / ((double)n_phi * P)));
            }
            w[(size_t)j * pp + p] = d;
        }
        return;
    }
    b -= n_a;
    const int q = 64 * b + lane;
    if (q >= (plan.n_c + 7) / 8 * 8) return;
    const int qn = min(q, plan.n_c - 1);   // up to a multiple of 8 the last node again
    int m = 0;
    while (plan.off[m + 1] <= qn) ++m;
    const double th = 0.5 * plan.theta_max * (1.0 + cheb_point(m, rows));
    const double rr = 2.0 * f * tan(0.5 * th);
    double s, c;
    sincospi(2.0 * (double)(qn - plan.off[m]) / (double)plan.cols[m], &s, &c);
    const double z = rr * rr / (4.0 * f), rs = z + f;   // |r_s| = r^2 / 4f + f on the paraboloid
    const double v[4] = {rr * c, rr * s, z - f, rs};
    for (int k = 0; k < 4; ++k) {
        if (pos64) pos64[4 * (size_t)q + k] = v[k];
        if (pos32) pos32[4 * (size_t)q + k] = (float)v[k];
    }
    if (hinv64) hinv64[q] = 0.5 / rs;
    if (dir32) {
        for (int k = 0; k < 3; ++k) dir32[4 * (size_t)q + k] = (float)(v[k] / rs);
        dir32[4 * (size_t)q + 3] = (float)(0.5 / rs);
    }
}

// One record (J~.x, J~.y, J~.z, rho~) from the tables an evaluation reads, general or factored (J~ = u s),
// in FP32 or FP64: the loads, and the 8 doubles made of them.
template <typename R>
struct RawRecord {
    typedef R r4 __attribute__((ext_vector_type(4)));
    r4 a, b;
};
template <typename R, bool FACT>
__device__ __forceinline__ RawRecord<R> load_record(const R *__restrict__ tab, const R *__restrict__ pos, int64_t rec,
                                                    int64_t node)
{
    typedef typename RawRecord<R>::r4 r4;
    if constexpr (FACT) return {*(const r4 *)(tab + rec * 4), *(const r4 *)(pos + node * 8 + 4)};
    else return {*(const r4 *)(tab + rec * 8), *(const r4 *)(tab + rec * 8 + 4)};
}
template <typename R, bool FACT>
__device__ __forceinline__ void record_doubles(const RawRecord<R> &r, double *v)
{
    if constexpr (FACT) {
        const double x = (double)r.a.x, y = (double)r.a.y;
        v[0] = (double)r.b.x * x;
        v[1] = (double)r.b.x * y;
        v[2] = (double)r.b.y * x;
        v[3] = (double)r.b.y * y;
        v[4] = (double)r.b.z * x;
        v[5] = (double)r.b.z * y;
        v[6] = (double)r.a.z;
        v[7] = (double)r.a.w;
    } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            v[c] = (double)r.a[c];
            v[4 + c] = (double)r.b[c];
        }
    }
}

// The contraction over the radii: one wave per (frequency, part of the radii, 16 phi, 16 rows), 8
// accumulators of 16 x 16 (one per real of the record).  Waves are numbered with the row tiles fastest,
// so that neighbours read the same records, four to a workgroup, and load ROWS_DEPTH steps ahead.  Bound
// by the FP64 pipe: the matrix instructions take 64 cycles each, and the conversion of a record (14
// FP64 instructions) runs on the same pipe and is not hidden behind them: 41 rows, 128 frequencies and
// 160 400 nodes take 0.32 ms, 50 TFLOP/s of matrix work (a large FP64 product on this card: 69).  The
// waves-per-SIMD request keeps the accumulators in plain registers: without it the compiler moved all 64
// through accumulation registers in every step (80 of 119 instructions), 0.41 ms.  Two or three row
// tiles per wave, so that a record is converted once for them, took 0.40 and 0.32 ms.
constexpr int ROWS_DEPTH = 2;
template <typename R, bool FACT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
k_compact_rows(int k0, int n_r, int n_phi, int rows, int split, int64_t n_waves, const R *__restrict__ tab,
               const R *__restrict__ pos, const double *__restrict__ wrad, double *__restrict__ T)
{
    const int lane = threadIdx.x & 63, kq = lane >> 4, col = lane & 15;
    const int groups = (n_phi + 15) / 16, rp = (rows + 15) / 16 * 16, tiles = rp / 16;
    const int64_t wave = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (wave >= n_waves) return;
    const int m0 = 16 * (int)(wave % tiles);
    const int64_t rest = wave / tiles;
    const int g = (int)(rest % groups), ks = (int)(rest / groups);
    const int part = ks % split, kk = ks / split;
    const int phi = 16 * g + col, ph = min(phi, n_phi - 1);
    const int n_i = n_r + 1, steps = (n_i + 3) / 4;
    const int s0 = (int)((int64_t)steps * part / split), s1 = (int)((int64_t)steps * (part + 1) / split);
    const int64_t rec0 = (int64_t)(k0 + kk) * n_i * n_phi;
    d4 acc[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[c] = d4{0.0, 0.0, 0.0, 0.0};
    RawRecord<R> raw[ROWS_DEPTH];
    double wgt[ROWS_DEPTH];
    auto load = [&](int d, int s) {
        const int i = 4 * min(s, s1 - 1) + kq;
        const int64_t node = (int64_t)min(i, n_r) * n_phi + ph;   // past the rim: weight 0
        wgt[d] = wrad[(size_t)i * rp + m0 + col];
        raw[d] = load_record<R, FACT>(tab, pos, rec0 + node, node);
    };
    auto step = [&](int d, int s) {
        double v[8];
        record_doubles<R, FACT>(raw[d], v);
        const double a = wgt[d];
        load(d, s + ROWS_DEPTH);
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, v[c], acc[c], 0, 0, 0);
    };
#pragma unroll
    for (int d = 0; d < ROWS_DEPTH; ++d) load(d, s0 + d);
    int s = s0;
    for (; s + ROWS_DEPTH <= s1; s += ROWS_DEPTH) {
#pragma unroll
        for (int d = 0; d < ROWS_DEPTH; ++d) step(d, s + d);
    }
#pragma unroll
    for (int d = 0; d < ROWS_DEPTH - 1; ++d)
        if (s + d < s1) step(d, s + d);
    if (phi >= n_phi) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int m = m0 + 4 * q + kq;
        if (m >= rows) continue;
        d2 *dst = (d2 *)(T + (((size_t)ks * rows + m) * n_phi + phi) * 8);
#pragma unroll
        for (int c = 0; c < 4; ++c) dst[c] = d2{acc[2 * c][q], acc[2 * c + 1][q]};
    }
}

constexpr int COLS_KP = 4;   // pairs of frequencies per wave

// The contraction over phi: one workgroup per (row, 16 columns, 8 frequencies), its four waves each a
// quarter of the phi, joined in LDS in a fixed order; the 16 columns of a product are 2 frequencies x 8
// reals, and the angular weights serve the 4 products of a wave.  Latency of the T loads is what
// bounds it: with one wave for all phi and two steps in flight it took 135 us at 128 frequencies and
// 130-200 us at 5 to 30, where there are few workgroups.
template <typename OT, bool SPLIT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
k_compact_cols(CompactPlan plan, int n_k, int n_phi, const double *__restrict__ wang, const double *__restrict__ T,
               OT *__restrict__ out)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, kq = lane >> 4, col = lane & 15, c = col & 7;
    const int rows = plan.rows, split = plan.split;
    const int b = blockIdx.x;
    int m = 0;
    while (plan.poff[m + 1] <= 16 * b) ++m;
    const int P = plan.cols[m], p0 = 16 * b - plan.poff[m], pp = (P + 15) / 16 * 16;
    const double *w = wang + (size_t)plan.poff[m] * n_phi + p0 + col;
    const int kbase = blockIdx.y * 2 * COLS_KP + (col >> 3);
    const double *src[COLS_KP];
#pragma unroll
    for (int g = 0; g < COLS_KP; ++g)
        src[g] = T + ((size_t)min(kbase + 2 * g, n_k - 1) * split * rows + m) * n_phi * 8 + c;
    const size_t pstride = (size_t)rows * n_phi * 8;
    d4 acc[COLS_KP];
#pragma unroll
    for (int g = 0; g < COLS_KP; ++g) acc[g] = d4{0.0, 0.0, 0.0, 0.0};
    const int steps = (n_phi + 3) / 4, s0 = steps * wave / 4, s1 = steps * (wave + 1) / 4;
#pragma unroll 4
    for (int js = s0; js < s1; ++js) {
        const int j0 = 4 * js, j = min(j0 + kq, n_phi - 1);
        const double a = j0 + kq < n_phi ? w[(size_t)j * pp] : 0.0;
#pragma unroll
        for (int g = 0; g < COLS_KP; ++g) {
            double v = src[g][(size_t)j * 8];
            if constexpr (SPLIT)
                for (int s = 1; s < split; ++s) v += src[g][s * pstride + (size_t)j * 8];
            acc[g] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, v, acc[g], 0, 0, 0);
        }
    }
    __shared__ d4 part[3][COLS_KP][64];
    if (wave > 0) {
#pragma unroll
        for (int g = 0; g < COLS_KP; ++g) part[wave - 1][g][lane] = acc[g];
    }
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int g = 0; g < COLS_KP; ++g) {
        const int k = kbase + 2 * g;
        acc[g] = ((acc[g] + part[0][g][lane]) + part[1][g][lane]) + part[2][g][lane];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int p = p0 + 4 * q + kq;
            if (k < n_k && p < P) out[((size_t)k * plan.n_c + plan.off[m] + p) * 8 + c] = (OT)acc[g][q];
        }
    }
}

// ================================================================== launchers

hipError_t launch_compact_geometry(hipStream_t st, const CompactPlan &plan, int n_r, int n_phi, double f,
                                   const double *r, double *wrad, double *wang, int is_f64, void *pos, void *hinv)
{
    const int blocks = (n_r + 4) / 4 * 4 + plan.poff[plan.rows] / 16 * ((n_phi + GEOM_PHI - 1) / GEOM_PHI) +
                       (plan.n_c + 63) / 64;
    hipLaunchKernelGGL(k_compact_geometry, dim3(blocks), dim3(64), 0, st, plan, n_r, n_phi, f, r, wrad, wang,
                       is_f64 ? (double *)pos : nullptr, is_f64 ? (double *)hinv : nullptr,
                       is_f64 ? nullptr : (float *)pos, is_f64 ? nullptr : (float *)hinv);
    return hipGetLastError();
}

hipError_t launch_compact_tables(hipStream_t st, const CompactPlan &plan, int n_r, int n_phi, int k0, int n_k,
                                 int is_f64, int fact, const void *tab, const void *pos, const double *wrad,
                                 const double *wang, double *T, void *out)
{
    const int64_t n_waves = (int64_t)((plan.rows + 15) / 16) * ((n_phi + 15) / 16) * plan.split * n_k;
    const dim3 gr((unsigned)((n_waves + 3) / 4)), br(256);
#define SC_COMPACT_ROWS(R, F)                                                                                 \
    hipLaunchKernelGGL((k_compact_rows<R, F>), gr, br, 0, st, k0, n_r, n_phi, plan.rows, plan.split, n_waves, \
                       (const R *)tab, (const R *)pos, wrad, T)
    if (is_f64 && fact) SC_COMPACT_ROWS(double, true);
    else if (is_f64) SC_COMPACT_ROWS(double, false);
    else if (fact) SC_COMPACT_ROWS(float, true);
    else SC_COMPACT_ROWS(float, false);
#undef SC_COMPACT_ROWS
    const dim3 gc(plan.poff[plan.rows] / 16, (n_k + 2 * COLS_KP - 1) / (2 * COLS_KP));
#define SC_COMPACT_COLS(R, S) \
    hipLaunchKernelGGL((k_compact_cols<R, S>), gc, dim3(256), 0, st, plan, n_k, n_phi, wang, T, (R *)out)
    if (is_f64 && plan.split > 1) SC_COMPACT_COLS(double, true);
    else if (is_f64) SC_COMPACT_COLS(double, false);
    else if (plan.split > 1) SC_COMPACT_COLS(float, true);
    else SC_COMPACT_COLS(float, false);
#undef SC_COMPACT_COLS
    return hipGetLastError();
}

}  // namespace sc
