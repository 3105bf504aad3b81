// sc_compact.hip -- the compacted tables of a mirror's sum (see sc_compact.h), on the FP64 matrix
// instructions: c~ = (trigonometric interpolation)^T (Chebyshev interpolation)^T c per frequency.
//
//  k_compact_geometry   interpolation weights and the compacted nodes' records
//  k_compact_rows       T[m][phi] = sum_i L_m(theta_i) c[i][phi] + L_-m(theta_i) c[i][phi + pi]
//                                                                       (contraction over the radii)
//  k_compact_cols       c~[m][p]  = sum_j D_m(phi_j - psi_p) T[m][phi_j] (contraction over phi)
// With an odd n_phi phi + pi is no grid point, and T keeps its two terms apart (rows m and rows + m), which
// k_compact_cols joins with weights of their own.
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

// The row that x belongs to: start[m] <= x < start[m + 1].
__device__ __forceinline__ int row_of(const int32_t *start, int rows, int x)
{
    int lo = 0, hi = rows - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (start[mid] <= x) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Blocks of 64: first one per radius (radial weights), then the angular weights (one block per (16
// columns of a row, 64 phi)), then the compacted nodes.  Latency of a few sines each: 1.1e6 angular
// weights (400 phi, 2 700 nodes) took 67 us with one block for all phi of 16 columns.
constexpr int GEOM_PHI = 64;
__global__ void __launch_bounds__(64)
k_compact_geometry(CompactPlan plan, int n_r, int n_phi, double f, const double *__restrict__ r,
                   double *__restrict__ wrad, double *__restrict__ wang, double *__restrict__ pos64,
                   double *__restrict__ hinv64, float *__restrict__ pos32, float *__restrict__ dir32)
{
    const int lane = threadIdx.x, rows = plan.rows, stride = compact_radial_stride(plan);
    const int n_j = plan.fold ? n_phi : 2 * n_phi;
    const int n_i = (n_r + 4) / 4 * 4, n_g = (n_j + GEOM_PHI - 1) / GEOM_PHI, n_a = plan.woff[rows] / 16 * n_g;
    int b = blockIdx.x;
    if (b < n_i) {
        // barycentric weights of the 2 rows Chebyshev points: w_j = (-1)^j sin((2j + 1) pi / 4 rows), and those
        // of -x_j are the negative ones
        const double x = b <= n_r ? sin(plan.beta * (2.0 * atan(r[b] / (2.0 * f)) / plan.theta_max)) / plan.alpha : 0.0;
        double sum = 0.0;
        int hit = -1;
        for (int j = lane; j < rows; j += 64) {
            const double xj = cheb_point(j, 2 * rows), d = (x - xj) * (x + xj);
            if (d == 0.0) hit = j;
            const double w = sinpi((double)(2 * j + 1) / (double)(4 * rows));
            sum += (d == 0.0 ? 0.0 : ((j & 1) ? -w : w) * xj / d);
        }
        for (int o = 32; o > 0; o >>= 1) {
            sum += __shfl_xor(sum, o);
            hit = max(hit, __shfl_xor(hit, o));
        }
        sum *= 2.0;
        double *out = wrad + (size_t)b * stride;
        for (int j = lane; j < stride; j += 64) {
            // row, and whether this is the odd part (L_-m)
            const int half = plan.fold ? stride / 2 : rows, odd = j >= half, m = odd ? j - half : j;
            double l = 0.0;
            if (b <= n_r && m < rows) {
                const double xj = cheb_point(m, 2 * rows), d = (x - xj) * (x + xj);
                const double w = sinpi((double)(2 * m + 1) / (double)(4 * rows)), c = ((m & 1) ? -w : w) / sum;
                if (plan.fold) l = hit >= 0 ? (m == hit ? 0.5 : 0.0) : c * (odd ? x : xj) / d;
                else if (hit >= 0) l = m == hit && !odd ? 1.0 : 0.0;
                else l = odd ? -c / (x + xj) : c / (x - xj);
            }
            out[j] = l;
        }
        return;
    }
    b -= n_i;
    if (b < n_a) {
        const int pt = b / n_g, j0 = (b - pt * n_g) * GEOM_PHI, j1 = min(j0 + GEOM_PHI, n_j);
        const int m = row_of(plan.woff, rows, 16 * pt);
        const int P = plan.cols[m], p0 = 16 * pt - plan.woff[m], pp = angular_kept(P);
        double *w = wang + (size_t)plan.woff[m] * n_j;
        const int p = p0 + (lane & 15);
        for (int jj = j0 + (lane >> 4); jj < j1; jj += 4) {
            double d = 0.0;
            if (p < P) {
                // sin(P x / 2) / (P sin(x / 2)) at x = 2 pi (j / n_phi - p / P), + pi for theta < 0, on exact integers
                // (the plan keeps n_j P below 16e6)
                const int j = jj < n_phi ? jj : jj - n_phi;
                const int np = n_phi * P, a = 2 * (j * P - p * n_phi) + (jj < n_phi ? 0 : np);
                if (a == 0 || a == 2 * np) d = 1.0;
                else if (P < n_j)
                    d = sinpi((double)(a % (4 * n_phi)) / (double)(2 * n_phi)) /
                        (P * sinpi((double)a / (2.0 * (double)np)));
            }
            w[(size_t)jj * pp + p] = d;
        }
        return;
    }
    b -= n_a;
    const int q = 64 * b + lane;
    if (q >= (plan.n_c + 7) / 8 * 8) return;
    const int qn = min(q, plan.n_c - 1);   // up to a multiple of 8 the last node again
    const int m = row_of(plan.off, rows, qn);
    const double th = plan.theta_max * (asin(plan.alpha * cheb_point(m, 2 * rows)) / plan.beta);
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
// accumulators of 16 x 16 (one per real of the record).  FOLD: with E and O the even and odd part of L_m
// in theta, L_m c[phi] + L_-m c[phi + pi] = E (c[phi] + c[phi + pi]) + O (c[phi] - c[phi + pi]), and at
// phi + pi the same with - O: two sets of accumulators over half the phi, half the products of the two
// terms apart.  Waves are numbered with the row tiles fastest, so that neighbours read the same records,
// four to a workgroup, and load ROWS_DEPTH steps ahead.  Bound by the FP64 pipe: the matrix
// instructions take 64 cycles each, and the conversion of a record (14 FP64 instructions) runs on the same
// pipe and is not hidden behind them: 25 rows (32 with the padding), 128 frequencies and 160 400 nodes take
// 0.26 ms, 40 TFLOP/s of matrix work (a large FP64 product on this card: 69).  The waves-per-SIMD request keeps the accumulators in plain
// registers: without it the compiler moved them through accumulation registers in every step (80 of 119
// instructions, 0.41 ms for 0.32 without FOLD at 41 rows).
constexpr int ROWS_DEPTH = 2;
template <typename R, bool FACT, bool FOLD>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(FOLD ? 2 : 4)))
k_compact_rows(int k0, int n_r, int n_phi, int rows, int split, int64_t n_waves, const R *__restrict__ tab,
               const R *__restrict__ pos, const double *__restrict__ wrad, double *__restrict__ T)
{
    constexpr int S = FOLD ? 2 : 1;
    const int lane = threadIdx.x & 63, kq = lane >> 4, col = lane & 15;
    const int phis = FOLD ? n_phi / 2 : n_phi;   // of the waves; FOLD: each with phi + pi
    const int groups = (phis + 15) / 16, rp = (rows + 15) / 16 * 16, tiles = rp / 16;
    const int64_t wave = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (wave >= n_waves) return;
    const int m0 = 16 * (int)(wave % tiles);
    const int64_t rest = wave / tiles;
    const int g = (int)(rest % groups), ks = (int)(rest / groups);
    const int part = ks % split, kk = ks / split;
    const int phi = 16 * g + col, ph = min(phi, phis - 1);
    const int n_i = n_r + 1, steps = (n_i + 3) / 4;
    const int s0 = (int)((int64_t)steps * part / split), s1 = (int)((int64_t)steps * (part + 1) / split);
    const int64_t rec0 = (int64_t)(k0 + kk) * n_i * n_phi;
    d4 acc[S][8];
#pragma unroll
    for (int e = 0; e < S; ++e)
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[e][c] = d4{0.0, 0.0, 0.0, 0.0};
    RawRecord<R> raw[ROWS_DEPTH][S];
    double wgt[ROWS_DEPTH][S];
    auto load = [&](int d, int s) {
        const int i = 4 * min(s, s1 - 1) + kq;
        const int64_t node = (int64_t)min(i, n_r) * n_phi + ph;   // past the rim: weight 0
#pragma unroll
        for (int e = 0; e < S; ++e) {
            wgt[d][e] = wrad[((size_t)i * S + e) * rp + m0 + col];
            raw[d][e] = load_record<R, FACT>(tab, pos, rec0 + node + e * phis, node + e * phis);
        }
    };
    auto step = [&](int d, int s) {
        double v[S][8], a[S];
#pragma unroll
        for (int e = 0; e < S; ++e) {
            record_doubles<R, FACT>(raw[d][e], v[e]);
            a[e] = wgt[d][e];
        }
        load(d, s + ROWS_DEPTH);
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            if constexpr (FOLD) {
                const double sum = v[0][c] + v[1][c], dif = v[0][c] - v[1][c];
                acc[0][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[0], sum, acc[0][c], 0, 0, 0);
                acc[1][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[1], dif, acc[1][c], 0, 0, 0);
            } else {
                acc[0][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[0], v[0][c], acc[0][c], 0, 0, 0);
            }
        }
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
    if (phi >= phis) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int m = m0 + 4 * q + kq;
        if (m >= rows) continue;
        d2 *dst = (d2 *)(T + (((size_t)ks * rows + m) * n_phi + phi) * 8);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const d2 x = {acc[0][2 * c][q], acc[0][2 * c + 1][q]};
            if constexpr (FOLD) {
                const d2 y = {acc[S - 1][2 * c][q], acc[S - 1][2 * c + 1][q]};
                dst[c] = x + y;
                dst[c + 4 * phis] = x - y;
            } else {
                dst[c] = x;
            }
        }
    }
}

constexpr int COLS_KP = 4;   // pairs of frequencies per wave

// The contraction over phi: one workgroup per (row, 16 columns, 8 frequencies), its four waves each a
// quarter of the phi, joined in LDS in a fixed order; the 16 columns of a product are 2 frequencies x 8
// reals, and the angular weights serve the 4 products of a wave.  Latency of the T loads is what
// bounds it: with one wave for all phi and two steps in flight it took 135 us at 128 frequencies (41 rows,
// not folded; now 73 us, 25 rows) and 130-200 us at 5 to 30, where there are few workgroups.
// (SP: the radii's parts, rounded up to a power of two; they are loaded together and added, past the last
// one that one again.  One after the other took 48 us for 5 parts at 12 frequencies.)
template <typename OT, int SP, bool FOLD>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
k_compact_cols(CompactPlan plan, int n_k, int n_phi, const double *__restrict__ wang, const double *__restrict__ T,
               OT *__restrict__ out)
{
    constexpr int S = FOLD ? 1 : 2;   // terms of T that are apart
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, kq = lane >> 4, col = lane & 15, c = col & 7;
    const int rows = plan.rows, split = plan.split;
    const int b = blockIdx.x;
    const int m = row_of(plan.poff, rows, 16 * b);
    const int P = plan.cols[m], p0 = 16 * b - plan.poff[m], pp = angular_kept(P);
    // a column beyond half reads its mirror image at -phi (one beyond P, never stored, the first)
    const int p = p0 + col;
    const bool mirror = p < P && p > P / 2;
    const double *w = wang + (size_t)plan.woff[m] * (S * n_phi) + (p >= P ? 0 : mirror ? P - p : p);
    const int kbase = blockIdx.y * 2 * COLS_KP + (col >> 3);
    const double *src[COLS_KP];
    const size_t pstride = (size_t)S * rows * n_phi * 8;
#pragma unroll
    for (int g = 0; g < COLS_KP; ++g)
        src[g] = T + (size_t)min(kbase + 2 * g, n_k - 1) * split * pstride + (size_t)m * n_phi * 8 + c;
    d4 acc[COLS_KP];
#pragma unroll
    for (int g = 0; g < COLS_KP; ++g) acc[g] = d4{0.0, 0.0, 0.0, 0.0};
    const int steps = (n_phi + 3) / 4, s0 = steps * wave / 4, s1 = steps * (wave + 1) / 4;
#pragma unroll
    for (int e = 0; e < S; ++e) {
        const double *we = w + (size_t)e * n_phi * pp;
        const size_t off = (size_t)e * rows * n_phi * 8;
#pragma unroll 4
        for (int js = s0; js < s1; ++js) {
            const int j0 = 4 * js, j = min(j0 + kq, n_phi - 1);
            const double a = j0 + kq < n_phi ? we[(size_t)(mirror && j ? n_phi - j : j) * pp] : 0.0;
#pragma unroll
            for (int g = 0; g < COLS_KP; ++g) {
                double part[SP];
#pragma unroll
                for (int s = 0; s < SP; ++s) part[s] = src[g][off + min(s, split - 1) * pstride + (size_t)j * 8];
                double v = part[0];
#pragma unroll
                for (int s = 1; s < SP; ++s) v += s < split ? part[s] : 0.0;
                acc[g] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, v, acc[g], 0, 0, 0);
            }
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
            const int po = p0 + 4 * q + kq;
            if (k < n_k && po < P) out[((size_t)k * plan.n_c + plan.off[m] + po) * 8 + c] = (OT)acc[g][q];
        }
    }
}

// ================================================================== launchers

hipError_t launch_compact_geometry(hipStream_t st, const CompactPlan &plan, int n_r, int n_phi, double f,
                                   const double *r, double *wrad, double *wang, int is_f64, void *pos, void *hinv)
{
    const int n_j = plan.fold ? n_phi : 2 * n_phi;
    const int blocks = (n_r + 4) / 4 * 4 + plan.woff[plan.rows] / 16 * ((n_j + GEOM_PHI - 1) / GEOM_PHI) +
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
    // without the fold the rows of theta < 0 are summed as rows of their own
    const int rows = plan.fold ? plan.rows : 2 * plan.rows, phis = plan.fold ? n_phi / 2 : n_phi;
    const int64_t n_waves = (int64_t)((rows + 15) / 16) * ((phis + 15) / 16) * plan.split * n_k;
    const dim3 gr((unsigned)((n_waves + 3) / 4)), br(256);
    const dim3 gc(plan.poff[plan.rows] / 16, (n_k + 2 * COLS_KP - 1) / (2 * COLS_KP));
#define SC_COMPACT_ROWS(R, F, FO)                                                                              \
    hipLaunchKernelGGL((k_compact_rows<R, F, FO>), gr, br, 0, st, k0, n_r, n_phi, rows, plan.split, n_waves,   \
                       (const R *)tab, (const R *)pos, wrad, T)
#define SC_COMPACT_COLS(R, S, FO) \
    hipLaunchKernelGGL((k_compact_cols<R, S, FO>), gc, br, 0, st, plan, n_k, n_phi, wang, T, (R *)out)
#define SC_COMPACT(R, FO)                                     \
    do {                                                      \
        if (fact) SC_COMPACT_ROWS(R, true, FO);               \
        else SC_COMPACT_ROWS(R, false, FO);                   \
        if (plan.split > 4) SC_COMPACT_COLS(R, 8, FO);        \
        else if (plan.split > 2) SC_COMPACT_COLS(R, 4, FO);   \
        else if (plan.split > 1) SC_COMPACT_COLS(R, 2, FO);   \
        else SC_COMPACT_COLS(R, 1, FO);                       \
    } while (0)
    if (is_f64 && plan.fold) SC_COMPACT(double, true);
    else if (is_f64) SC_COMPACT(double, false);
    else if (plan.fold) SC_COMPACT(float, true);
    else SC_COMPACT(float, false);
#undef SC_COMPACT
#undef SC_COMPACT_COLS
#undef SC_COMPACT_ROWS
    return hipGetLastError();
}

}  // namespace sc
