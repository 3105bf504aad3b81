// sc_quad_mm.hip -- the quadrature over compacted nodes in the FP32 split form, its contraction on the
// FP16 matrix instructions.
//
// With G = e^{ik delta} / R and H = (ik - 1/R) G / R of a node and a point, R_vec = r_s - r',
//   E  = sum G J~ + H rho~ r_s - r' sum H rho~
//   B' = sum H (J~ x r_s) - (sum H J~) x r'
// so the kernel values G and H (four reals per node, point and frequency) meet ten complex columns
// of table data that do not depend on the point: a matrix product.  The vector ALU forms G and H (one
// phase, one sine, one cosine, 7 more instructions) and v_mfma_f32_32x32x16_f16 sums them over the
// nodes, where the plain form spends 47 more FMAs per term on the vector ALU.
//
// Precision.  Every kernel value and every table entry of E and B is the sum of two FP16 numbers,
// hi = fp16(x) and lo = fp16(x - hi): 22 bits, and all four products of the parts are summed in FP32
// (rows of A: hi and lo of the table; two products per step: hi and lo of the kernel values).  The
// columns that r' multiplies (|r'| <= |r_s| / 4) are hi alone where |r'| <= |r_s| / 100, and get
// their lo part by a third product otherwise.  Table columns are scaled by powers of two to 2^12 at
// most, and the kernel values to about 2^6, so that no lo part falls below FP16's smallest number.
// Against 64 bits the sums are as exact as the plain FP32 form's: broadband 4.2e-7 (plain 4.2e-7).
//
// One step is 4 nodes: lane l holds point l % 32 and nodes 2 (l / 32), 2 (l / 32) + 1 of the step as B's
// 8 consecutive values (Gr, Gi, Hr, Hi of each), and row l % 32 of A, 16 B loaded as they lie.
#include "sc_device.h"
#include "sc_internal.h"

namespace sc {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(4))) const QuadJob cjob;
typedef __attribute__((address_space(4))) const double cdouble;
typedef __attribute__((address_space(4))) const float cfloat;

// Kernel values are formed as G s * 2^6 and H s^2 / k * 2^6 with s a power of two near the focal length.
constexpr float KERNEL_SCALE = 64.0f;

// v = hi + lo to 22 bits; m1 is -1 from memory, so that the difference is one mixed-precision FMA.
__device__ __forceinline__ void split2(float a, float b, float m1, h2 &hi, h2 &lo)
{
    const v2f v = {a, b};
    hi = __builtin_convertvector(v, h2);
    const v2f l = {__builtin_fmaf((float)hi.x, m1, a), __builtin_fmaf((float)hi.y, m1, b)};
    lo = __builtin_convertvector(l, h2);
}

template <int F, bool RAW, bool SER, bool FAR>
__device__ __forceinline__ void tile_mm(cjob *job, int chunk, int pg, int kb, float m1)
{
    const int lane = threadIdx.x & 63, half = lane >> 5;
    const int n_k = job->n_k, n_obs_pad = job->n_obs_pad, steps = (job->n_tot + 3) / 4;
    const int s0 = chunk * (job->chunk / 4), s1 = min(s0 + job->chunk / 4, steps);
    const int pt = pg * 128 + (threadIdx.x >> 6) * 32 + (lane & 31);
    const float s = job->scale;
    float kt[F], iks[F];
    const h8 *A[F];
    const size_t row = (size_t)steps * 64;
#pragma unroll
    for (int f = 0; f < F; ++f) {
        const int k = min(kb * F + f, n_k - 1);
        const double kv = ((cdouble *)job->k)[k];
        kt[f] = (float)(kv * INV_TWO_PI);
        iks[f] = (float)(1.0 / (kv * (double)s));
        A[f] = (const h8 *)job->mtab + (size_t)k * (FAR ? 2 : 1) * row + lane;
    }
    const v4f o = ((const v4f *)job->obs)[pt];
    const v4f *pos = (const v4f *)job->pos;
    const float *hinv = (const float *)job->hinv;
    v16f acc[F];
#pragma unroll
    for (int f = 0; f < F; ++f)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[f][v] = 0.0f;

    for (int st = s0; st < s1; ++st) {
        const int n = 4 * st + 2 * half;
        float ph[2], delta[2];   // s / R and |R| - |r_s|
        const v2f h = *(const v2f *)(hinv + n);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const v4f p = pos[n + q];
            const float dot = __fmaf_rn(p.x, o.x, __fmaf_rn(p.y, o.y, p.z * o.z));
            const float num = __fmaf_rn(-2.0f, dot, o.w);
            if constexpr (SER) {   // series near the focus, as in the plain form
                const float hq = q ? h.y : h.x;
                const float d1 = num * hq, x = d1 * hq;
                delta[q] = d1 * __fmaf_rn(x, __fmaf_rn(2.0f, x, -1.0f), 1.0f);
                const float h2s = hq + hq, y = delta[q] * h2s;
                ph[q] = (h2s * s) * __fmaf_rn(y, y - 1.0f, 1.0f);
            } else {
                const float dx = p.x - o.x, dy = p.y - o.y, dz = p.z - o.z;
                const float R2 = __fmaf_rn(dx, dx, __fmaf_rn(dy, dy, dz * dz));
                const float rinv = __builtin_amdgcn_rsqf(R2);
                delta[q] = num * __builtin_amdgcn_rcpf(__fmaf_rn(R2, rinv, p.w));
                ph[q] = rinv * s;
            }
        }
#pragma unroll
        for (int f = 0; f < F; ++f) {
            const h8 a = A[f][(size_t)st * 64];
            h2 hi[4], lo[4];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const float turn = kt[f] * delta[q];
                const float r = RAW ? turn : __builtin_amdgcn_fractf(turn);
                const float pa = ph[q] * KERNEL_SCALE;
                const float gr = __builtin_amdgcn_cosf(r) * pa, gi = __builtin_amdgcn_sinf(r) * pa;
                const float b = (ph[q] * ph[q]) * iks[f];
                // H s^2 / k = (i s / R - (s / R)^2 / (k s)) G s
                const float hr = -__fmaf_rn(gi, ph[q], gr * b), hi_ = __fmaf_rn(gr, ph[q], -(gi * b));
                split2(gr, gi, m1, hi[2 * q], lo[2 * q]);
                split2(hr, hi_, m1, hi[2 * q + 1], lo[2 * q + 1]);
            }
            const h8 bh = {hi[0].x, hi[0].y, hi[1].x, hi[1].y, hi[2].x, hi[2].y, hi[3].x, hi[3].y};
            const h8 bl = {lo[0].x, lo[0].y, lo[1].x, lo[1].y, lo[2].x, lo[2].y, lo[3].x, lo[3].y};
            acc[f] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, bh, acc[f], 0, 0, 0);
            if constexpr (FAR)
                acc[f] = __builtin_amdgcn_mfma_f32_32x32x16_f16(A[f][row + (size_t)st * 64], bh, acc[f], 0, 0, 0);
            acc[f] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, bl, acc[f], 0, 0, 0);
        }
    }
    // Rows of a lane: lanes 0-31 E hi (6), E lo (6), sum H rho~ (2), (sum H J~).z (2); lanes 32-63 B hi, B lo,
    // (sum H J~).x, .y
    const float ox = o.x, oy = o.y, oz = o.z;
#pragma unroll
    for (int f = 0; f < F; ++f) {
        const int k = kb * F + f;
        float jzr = __shfl_xor(acc[f][14], 32), jzi = __shfl_xor(acc[f][15], 32);
        if (k >= n_k) continue;
        cfloat *sc = (cfloat *)job->mscale + 16 * (size_t)k;
        float v[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) v[c] = (acc[f][c] + acc[f][6 + c]) * (half ? sc[4 + c / 2] : sc[c / 2]);
        if (half == 0) {
            const float sr = acc[f][12] * sc[3], si = acc[f][13] * sc[3];
            v[0] = __fmaf_rn(-sr, ox, v[0]);
            v[1] = __fmaf_rn(-si, ox, v[1]);
            v[2] = __fmaf_rn(-sr, oy, v[2]);
            v[3] = __fmaf_rn(-si, oy, v[3]);
            v[4] = __fmaf_rn(-sr, oz, v[4]);
            v[5] = __fmaf_rn(-si, oz, v[5]);
        } else {
            const float jxr = acc[f][12] * sc[7], jxi = acc[f][13] * sc[7];
            const float jyr = acc[f][14] * sc[8], jyi = acc[f][15] * sc[8];
            jzr *= sc[9];
            jzi *= sc[9];
            v[0] -= __fmaf_rn(jyr, oz, -(jzr * oy));
            v[1] -= __fmaf_rn(jyi, oz, -(jzi * oy));
            v[2] -= __fmaf_rn(jzr, ox, -(jxr * oz));
            v[3] -= __fmaf_rn(jzi, ox, -(jxi * oz));
            v[4] -= __fmaf_rn(jxr, oy, -(jyr * ox));
            v[5] -= __fmaf_rn(jxi, oy, -(jyi * ox));
        }
        // partials [chunk][k][point / 64][12][64]
        float *part = (float *)job->partial + ((size_t)chunk * n_k + k) * 12 * (size_t)n_obs_pad + (size_t)(pt >> 6) * 768 +
                      half * 384 + (pt & 63);
#pragma unroll
        for (int c = 0; c < 6; ++c) part[c * 64] = v[c];
    }
}

// One workgroup per tile: 128 points (32 per wave) x F frequencies x one chunk of nodes, the four waves
// reading the same table rows through L1.  Tiles run points fastest; workgroups go to the 8 XCDs in turn,
// so each XCD takes a contiguous eighth of the tiles and its L2 serves the rows that they share.
// (job_tile: tile t of the launch, which is one of this job's.)
template <int F>
__device__ __forceinline__ void job_tile(cjob *job, int64_t t, float m1)
{
    const int64_t local = t - job->tile0 + job->tile_offset;
    const int pgs = job->n_obs_pad / 128;
    const int pg = (int)(local % pgs);
    const int64_t rest = local / pgs;
    const int chunk = (int)(rest % job->n_chunks), kb = (int)(rest / job->n_chunks);
    const bool raw = job->raw_phase != 0, ser = job->series_delta != 0;
    if (ser && raw) tile_mm<F, true, true, false>(job, chunk, pg, kb, m1);
    else if (ser) tile_mm<F, false, true, false>(job, chunk, pg, kb, m1);
    else if (!job->far) {
        if (raw) tile_mm<F, true, false, false>(job, chunk, pg, kb, m1);
        else tile_mm<F, false, false, false>(job, chunk, pg, kb, m1);
    } else {
        if (raw) tile_mm<F, true, false, true>(job, chunk, pg, kb, m1);
        else tile_mm<F, false, false, true>(job, chunk, pg, kb, m1);
    }
}

// The tiles of this workgroup: its XCD's eighth from its own place on.
#define SC_MM_TILES(t)                                                                              \
    const int64_t per = (n_tiles + QUAD_SEGMENTS - 1) / QUAD_SEGMENTS;                              \
    const int64_t end = min(n_tiles, per * (int64_t)(blockIdx.x % QUAD_SEGMENTS + 1));              \
    for (int64_t t = per * (int64_t)(blockIdx.x % QUAD_SEGMENTS) + blockIdx.x / QUAD_SEGMENTS; t < end; \
         t += gridDim.x / QUAD_SEGMENTS)

// One job, which travels as the kernel's first argument and is read where it lies.
template <int F>
__global__ void __launch_bounds__(256) k_quad_mm_one(QuadJob, int64_t n_tiles, float m1)
{
    cjob *job = (cjob *)__builtin_amdgcn_kernarg_segment_ptr();
    SC_MM_TILES(t) job_tile<F>(job, t, m1);
}

// Tiles of several jobs.
template <int F>
__global__ void __launch_bounds__(256)
k_quad_mm(const QuadJob *__restrict__ jobs_, int n_jobs, int64_t n_tiles, float m1)
{
    cjob *jobs = (cjob *)jobs_;
    SC_MM_TILES(t) {
        int lo = 0, hi = n_jobs - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (jobs[mid].tile0 <= t) lo = mid;
            else hi = mid - 1;
        }
        job_tile<F>(jobs + lo, t, m1);
    }
}

// ------------------------------------------------------------------------------- packed tables

// The ten complex columns of node q at wavenumber k, in the order of the scales: E.x, E.y, E.z as (g, h)
// pairs (G's factor J~ / s, H's factor k / s^2 rho~ r_s), then the H columns rho~, (J~ x r_s).x, .y, .z,
// J~.x, .y, .z times k / s^2.
__device__ __forceinline__ void mm_columns(const float *__restrict__ rec, const v4f p, double k, double s, double *g,
                                           double *h)
{
    const double js = 1.0 / s, hs = k / (s * s), r[3] = {p.x, p.y, p.z};
    double J[6], rho[2] = {hs * (double)rec[6], hs * (double)rec[7]};
    for (int c = 0; c < 6; ++c) {
        g[c] = js * (double)rec[c];
        J[c] = hs * (double)rec[c];
    }
    for (int z = 0; z < 2; ++z) {   // re, im
        for (int c = 0; c < 3; ++c) h[2 * c + z] = rho[z] * r[c];
        h[6 + z] = rho[z];
        h[8 + z] = J[2 + z] * r[2] - J[4 + z] * r[1];
        h[10 + z] = J[4 + z] * r[0] - J[z] * r[2];
        h[12 + z] = J[z] * r[1] - J[2 + z] * r[0];
        for (int c = 0; c < 3; ++c) h[14 + 2 * c + z] = J[2 * c + z];
    }
}

// Powers of two that bring each column's largest entry to 2^11 ... 2^12: mscale[k][16] holds what the
// sums are multiplied by (scale / KERNEL_SCALE).  One workgroup per frequency.
__global__ void __launch_bounds__(1024)
k_mm_scales(int n_c, const double *__restrict__ kv, double s, const float *__restrict__ ctab,
            const v4f *__restrict__ pos, float *__restrict__ mscale)
{
    const int kk = blockIdx.x;
    double mx[10] = {};
    for (int q = threadIdx.x; q < n_c; q += 1024) {
        double g[6], h[20];
        mm_columns(ctab + ((size_t)kk * n_c + q) * 8, pos[q], kv[kk], s, g, h);
        for (int c = 0; c < 10; ++c) {
            double m = fmax(fabs(h[2 * c]), fabs(h[2 * c + 1]));
            if (c < 3) m = fmax(m, fmax(fabs(g[2 * c]), fabs(g[2 * c + 1])));
            mx[c] = fmax(mx[c], m);
        }
    }
    __shared__ double red[16][10];
    for (int c = 0; c < 10; ++c) {
        double m = mx[c];
        for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o));
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][c] = m;
    }
    __syncthreads();
    if (threadIdx.x < 16) {
        double m = 0.0;
        if (threadIdx.x < 10)
            for (int w = 0; w < 16; ++w) m = fmax(m, red[w][threadIdx.x]);
        // m = f 2^e with f in [0.5, 1): times 2^(12 - e)
        const int e = m > 0.0 && m < 1e300 ? max(-100, min(100, ilogb(m) + 1)) : 12;
        mscale[16 * (size_t)kk + threadIdx.x] = (float)(ldexp(1.0, e - 12) / KERNEL_SCALE);
    }
}

// mtab[k][step][lane][8] halves: lane's row l % 32 of the two nodes 4 step + 2 (l / 32) + {0, 1}, for each the
// factors of (Gr, Gi, Hr, Hi); with `far` a second such table follows each frequency's, the lo
// parts of the columns that r' multiplies.  One wave per step.
__global__ void __launch_bounds__(256)
k_mm_pack(int n_c, int far, const double *__restrict__ kv, double s, const float *__restrict__ ctab,
          const v4f *__restrict__ pos, const float *__restrict__ mscale, h8 *__restrict__ mtab)
{
    const int steps = (n_c + 3) / 4, st = blockIdx.x * 4 + (threadIdx.x >> 6), kk = blockIdx.y;
    if (st >= steps) return;
    const int lane = threadIdx.x & 63, r = lane & 31, rh = (r >> 2) & 1, v = (r & 3) + 4 * (r >> 3);
    // row r holds value v of half rh (see tile_mm): its column, part (re, im) and whether it is the lo half
    int col, part = v & 1, lo = 0;
    if (v < 12) {
        lo = v >= 6;
        col = (rh ? 4 : 0) + (v % 6) / 2;
    } else if (rh == 0) {
        col = v < 14 ? 3 : 9;
    } else {
        col = v < 14 ? 7 : 8;
    }
    h8 out = {}, out2 = {};
    for (int q = 0; q < 2; ++q) {
        const int n = 4 * st + 2 * (lane >> 5) + q;
        if (n >= n_c) continue;   // past the last node: zero
        double g[6], h[20];
        mm_columns(ctab + ((size_t)kk * n_c + n) * 8, pos[n], kv[kk], s, g, h);
        const double inv = 1.0 / ((double)mscale[16 * (size_t)kk + col] * KERNEL_SCALE);   // a power of two
        double gr = 0.0, gi = 0.0, hr = 0.0, hi = 0.0;   // of this column
        for (int c = 0; c < 10; ++c)
            if (c == col) {
                hr = h[2 * c] * inv;
                hi = h[2 * c + 1] * inv;
                if (c < 3) {
                    gr = g[2 * c] * inv;
                    gi = g[2 * c + 1] * inv;
                }
            }
        // (a + ib)(Vr + iVi): re = a Vr - b Vi, im = b Vr + a Vi
        const float w[4] = {(float)(part ? gi : gr), (float)(part ? gr : -gi), (float)(part ? hi : hr),
                            (float)(part ? hr : -hi)};
        for (int e = 0; e < 4; ++e) {
            const _Float16 a = (_Float16)w[e], b = (_Float16)(w[e] - (float)a);
            out[4 * q + e] = lo ? b : a;
            if (v >= 12) out2[4 * q + e] = b;
        }
    }
    h8 *dst = mtab + ((size_t)kk * (far ? 2 : 1) * steps + st) * 64 + lane;
    dst[0] = out;
    if (far) dst[(size_t)steps * 64] = out2;
}

// ================================================================== launchers

hipError_t launch_mm_tables(hipStream_t st, int n_k, int n_c, int far, const double *k, double scale, const float *ctab,
                            const float *pos, float *mscale, void *mtab)
{
    hipLaunchKernelGGL(k_mm_scales, dim3(n_k), dim3(1024), 0, st, n_c, k, scale, ctab, (const v4f *)pos, mscale);
    hipLaunchKernelGGL(k_mm_pack, dim3(((n_c + 3) / 4 + 3) / 4, n_k), dim3(256), 0, st, n_c, far, k, scale, ctab,
                       (const v4f *)pos, mscale, (h8 *)mtab);
    return hipGetLastError();
}

static unsigned int mm_grid(int64_t n_tiles)
{
    const int64_t grid = (n_tiles + QUAD_SEGMENTS - 1) / QUAD_SEGMENTS * QUAD_SEGMENTS;
    return (unsigned int)(grid < (1 << 20) ? grid : (1 << 20));
}

hipError_t launch_quad_mm_one(hipStream_t st, int fpb, const QuadJob &job, int64_t n_tiles)
{
    const dim3 g(mm_grid(n_tiles)), b(256);
    if (fpb == 4) hipLaunchKernelGGL((k_quad_mm_one<4>), g, b, 0, st, job, n_tiles, -1.0f);
    else if (fpb == 2) hipLaunchKernelGGL((k_quad_mm_one<2>), g, b, 0, st, job, n_tiles, -1.0f);
    else hipLaunchKernelGGL((k_quad_mm_one<1>), g, b, 0, st, job, n_tiles, -1.0f);
    return hipGetLastError();
}

hipError_t launch_quad_mm(hipStream_t st, int fpb, const QuadJob *jobs, int n_jobs, int64_t n_tiles)
{
    const dim3 g(mm_grid(n_tiles)), b(256);
    if (fpb == 4) hipLaunchKernelGGL((k_quad_mm<4>), g, b, 0, st, jobs, n_jobs, n_tiles, -1.0f);
    else if (fpb == 2) hipLaunchKernelGGL((k_quad_mm<2>), g, b, 0, st, jobs, n_jobs, n_tiles, -1.0f);
    else hipLaunchKernelGGL((k_quad_mm<1>), g, b, 0, st, jobs, n_jobs, n_tiles, -1.0f);
    return hipGetLastError();
}

}  // namespace sc
